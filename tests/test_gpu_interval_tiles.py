"""The batched interval sweep at the edges of its tiles: interval counts that
leave rows unaligned or a last group of one to three, signal counts on both
sides of a tile and of a work-group's share, with and without gradients.
Every signal alone (the vector kernel) is the reference: both paths meet the
oracle's bounds of 1e-5 of the value, so they differ by at most twice that."""
import numpy as np
import pytest

from paper_2501_04194_amd import stl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,B,N", [(20, 16, 127), (20, 17, 4097), (20, 65, 16385), (5, 129, 131), (33, 81, 8194),
                                   (64, 16, 3)])
@pytest.mark.parametrize("grads", [True, False])
def test_sweep_tile_edges(T, B, N, grads):
    import torch
    rng = np.random.default_rng(T * B + N)
    x = torch.from_numpy(rng.uniform(-0.5, 0.5, size=(B, T, 1)).astype(np.float32)).cuda()
    a = torch.from_numpy(rng.uniform(-2.0, T, size=N).astype(np.float32)).cuda()
    b = a + torch.from_numpy(rng.uniform(0.5, T, size=N).astype(np.float32)).cuda()
    kw = dict(c=0.0, op="always", beta=10.0, mask_c=2.0, mask_eps=1e-6, grads=grads)
    scales = (1.0, 2.0 / 40, 2.0 / 40)       # rho; d/da, d/db: mask_c / (4 beta)

    def sweep(xs):
        r = stl.interval_sweep(xs, a, b, [1.0], **kw)
        return [v for v in (r if isinstance(r, (tuple, list)) else (r,)) if v is not None]

    got = sweep(x)
    for i in sorted({0, 1, B // 2, B - 2, B - 1}):
        for g, r, scale in zip(got, sweep(x[i:i + 1].contiguous()), scales):
            r = r.reshape(-1).double()
            bound = 2e-5 * (r.abs() + scale)
            bound[r.abs() == 1e6] = 0.0      # the empty-window value: exact
            assert bool(((g[i].double() - r).abs() <= bound).all()), (i, T, B, N)


@pytest.mark.parametrize("B,amp", [(65, 0.5), (79, 8.0)])
def test_sweep_large_batch_edges(B, amp):
    """Enough interval and signal tiles for four interval tiles per wave: ragged
    in both, and (amp = 8) sums that are redone against their own reference."""
    import torch
    T, N = 6, 256 * 13108 - 3
    rng = np.random.default_rng(B)
    x = torch.from_numpy(rng.uniform(-amp, amp, size=(B, T, 1)).astype(np.float32)).cuda()
    a = torch.from_numpy(rng.uniform(-2.0, T, size=N).astype(np.float32)).cuda()
    b = a + torch.from_numpy(rng.uniform(-0.5, T, size=N).astype(np.float32)).cuda()
    kw = dict(c=0.0, op="eventually", beta=10.0, mask_c=2.0, mask_eps=1e-6)
    got = stl.interval_sweep(x, a, b, [1.0], **kw)
    for i in (0, 15, B // 2, B - 2, B - 1):
        ref = stl.interval_sweep(x[i:i + 1].contiguous(), a, b, [1.0], **kw)
        for g, r, scale in zip(got, ref, (max(1.0, amp), 2.0 / 40, 2.0 / 40)):
            r = r.reshape(-1).double()
            bound = 2e-5 * (r.abs() + scale)
            bound[r.abs() == 1e6] = 0.0
            assert bool(((g[i].double() - r).abs() <= bound).all()), (i, B, amp)
