"""The one-launch descent on samples its FP32 terms cannot take: a signal with
a NaN or an infinity in the mask's support adds nothing to the loss and its
gradients, and terms far below a signal's largest one still count where that one
has a tiny weight.  The reference is the descent in 64-bit numpy; the bounds are
those of the other descent tests (2e-4 on the interval, 1e-4 of the loss)."""
import numpy as np
import pytest
import torch

from paper_2501_04194_amd import mining, stl

pytestmark = pytest.mark.gpu


def descent64(x, p, steps, lr, gamma, c_range, beta_range, op, eps):
    B, T = x.shape
    sg = 1.0 if op == "eventually" else -1.0
    k = np.arange(T, dtype=np.float64)
    p = p.astype(np.float64).copy()
    sig = lambda v: 1.0 / (1.0 + np.exp(-v))
    losses = []
    for i in range(steps):
        c, beta = mining.schedule(i, steps, *c_range), mining.schedule(i, steps, *beta_range)
        ab = sig(p)
        xa, xb = c * (k - ab[0] * T), c * (k - ab[1] * T)
        with np.errstate(over="ignore"):
            w = sig(xa) * sig(-xb) * -np.expm1(-c * (ab[1] - ab[0]) * T) - eps
            da, db = -c * sig(xa) * sig(-xa), c * sig(xb) * sig(-xb)
        on = w > 0.0
        loss, grad = 0.0, np.zeros(2)
        for row in x:
            z = sg * beta * row[on].astype(np.float64)
            if not np.isfinite(z).all():
                continue
            e = np.exp(z - z.max())
            S = (w[on] * e).sum()
            rho = sg * (z.max() + np.log(S)) / beta
            if rho < 0.0:
                loss -= rho
                grad -= sg / beta * np.array([(da[on] * e).sum(), (db[on] * e).sum()]) / S
        losses.append(loss / B + gamma * (ab[0] - ab[1]))
        p -= lr * (T * grad / B + np.array([gamma, -gamma])) * ab * (1.0 - ab)
    return p, np.array(losses)


def check(x, p0, steps, **kw):
    p = torch.from_numpy(p0).cuda()
    loss = stl.pstl_descent(torch.from_numpy(x[:, :, None].copy()).cuda(), p, steps, want_loss=True,
                            mask_eps=kw["eps"], **{k: v for k, v in kw.items() if k != "eps"}).cpu().numpy()
    rp, rl = descent64(x, p0, steps, **kw)
    p = p.cpu().numpy()
    assert np.isfinite(p).all() and np.isfinite(loss).all(), (p, loss)
    sig = lambda v: 1.0 / (1.0 + np.exp(-v))
    assert (np.abs(sig(p) - sig(rp)) < 2e-4).all(), (p, rp)
    assert (np.abs(loss - rl) <= 1e-4 * (1.0 + np.abs(rl))).all(), np.abs(loss - rl).max()


LOGITS = np.log(np.array([0.15, 0.8]) / np.array([0.85, 0.2])).astype(np.float32)


@pytest.mark.parametrize("op", ["always", "eventually"])
@pytest.mark.parametrize("B,T", [(40, 64), (500, 20), (1024, 12), (2000, 6)])
def test_nonfinite_signals_add_nothing(B, T, op):
    x = mining.make_dataset(B, T=T, seed=B)[:, :, 0] - (1.1 if op == "eventually" else 0.0)
    mid = T // 2
    for i, v in ((3, np.nan), (7, -np.inf), (11, np.inf)):
        x[i, mid] = v
        x[i + 12] = v
    check(x.astype(np.float32), LOGITS, 30, lr=1e-2, gamma=0.1, c_range=(2.0, 20.0), beta_range=(1.0, 20.0), op=op,
          eps=1e-6)


@pytest.mark.parametrize("op", ["always", "eventually"])
@pytest.mark.parametrize("B,T,c", [(1, 20, 10.0), (500, 20, 10.0), (1500, 8, 20.0)])
def test_terms_far_below_the_largest(B, T, c, op):
    """eps = 0: the signal's largest term lies 86 / c steps before the interval, where its weight is
    e^-86 = 2^-124; the interval's own terms are 2^-127 of it, a weight of about 1 each."""
    beta, k = 20.0, 1
    a = k + 86.0 / c
    sg = 1.0 if op == "eventually" else -1.0
    top = -1.0
    x = np.full((B, T), top - 40.0)
    x[:, k] = top
    x[:, int(np.ceil(a)):] = top - 127.0 * np.log(2.0) / beta
    b = min(a + 6.0, T - 0.1)
    logit = lambda v: np.log(v / (1.0 - v))
    p0 = np.array([logit(a / T), logit(b / T)], np.float32)
    x = (x if op == "eventually" else -x - 12.0).astype(np.float32)
    check(x, p0, 1, lr=1e-2, gamma=0.1, c_range=(c, c), beta_range=(beta, beta), op=op, eps=0.0)
