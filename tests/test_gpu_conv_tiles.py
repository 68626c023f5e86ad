"""The direct blur on the matrix cores (csrc/conv.hip) against the FP64 oracle
at the edges of its tiles: one and two products of depth 32 per row (p <= 25,
p > 25), 16-, 32- and 64-row tiles, ragged last tiles, every boundary model,
infinities and NaN.

Tolerance: with nonnegative data every output is a sum of nonnegative terms.
A product of the split parts misses at most 2^-24 of it, and the p + 1 row
products and their five corrections are summed in float32, one rounding (2^-24)
each, over one or two depths: 2 (p + 1) + 12 roundings at most.
"""
import numpy as np
import pytest
import torch

from oracle import blur as oblur
from paper_1504_07234_amd import mlba

pytestmark = pytest.mark.gpu


def _plan(n, p, bc, h):
    return mlba.Plan(n, p, bc, mlba.NONE, 1, torch.as_tensor(h, dtype=torch.float32).cuda())


def _data(n, p, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    h = g.uniform(0.0, 1.0, (p, p)) ** 4 + 1e-6
    h = (h / h.sum()).astype(np.float32).astype(np.float64)
    # four orders of magnitude, so that small values sit beside large ones
    y = (10.0 ** g.uniform(-4.0, 0.0, (n, n))).astype(np.float32).astype(np.float64)
    return h, y


CASES = [(n, p, bc) for n, p in ((15, 3), (16, 9), (17, 1), (63, 17), (64, 25), (65, 25), (49, 27), (64, 31), (127, 33),
                                 (130, 49)) for bc in range(5)]
CASES += [(770, 9, oblur.RECT), (1473, 5, oblur.REFLECT), (1500, 25, oblur.PERIODIC), (1030, 31, oblur.ZERO)]


@pytest.mark.parametrize("n,p,bc", CASES)
def test_adjoint_tiles(n, p, bc):
    h, y = _data(n, p, 100 * n + p)
    with _plan(n, p, bc, h) as plan:
        w = plan.apply_At(torch.as_tensor(y, dtype=torch.float32).cuda()).double().cpu().numpy()
    ref = oblur.blurT(y, h, bc, "direct" if n <= 130 else "auto")
    if bc == oblur.ANTIREFLECT:  # signed: relative to the largest value of the pad
        assert np.abs(w - ref).max() <= (2 * (p + 1) + 12) * 2.0 ** -24 * 3.0 * np.abs(y).max()
        return
    # the oracle's FFT form (large n) carries 1e-15 of the largest value; folds add at most four values
    tol = (2 * (p + 1) + 12 + 4) * 2.0 ** -24 * np.abs(ref) + 1e-14
    assert (np.abs(w - ref) <= tol).all(), np.abs(w - ref).max()


@pytest.mark.parametrize("n,p,bc", [(64, 9, oblur.RECT), (65, 25, oblur.REFLECT), (96, 31, oblur.ZERO),
                                    (97, 17, oblur.PERIODIC), (130, 33, oblur.ANTIREFLECT), (520, 15, oblur.RECT)])
def test_iteration_tiles(n, p, bc):
    """omega + A^T (g - A omega): P = I, no threshold, step 1 (W^T W = I)."""
    h, g = _data(n, p, 7 * n + p)
    N = n + p - 1 if bc == oblur.RECT else n
    omega = _data(N, 1, n)[1]
    with _plan(n, p, bc, h) as plan:
        z = torch.as_tensor(omega, dtype=torch.float32).cuda()
        plan.restore(torch.as_tensor(g, dtype=torch.float32).cuda(), mu=0.0, delta=1.0, iters=1, z=z, implicit=True)
        z = z.double().cpu().numpy()
    ref = omega + oblur.blurT(g - oblur.blur(omega, h, bc), h, bc)
    assert np.linalg.norm(z - ref) <= 1e-5 * np.linalg.norm(ref)


@pytest.mark.parametrize("n,p", [(70, 9), (70, 31)])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 3.4e38])
def test_not_finite(n, p, value):
    """Infinities and NaN reach exactly the outputs whose taps touch them."""
    h, y = _data(n, p, 3 * p)
    y[5, 60] = y[66, 3] = value
    with _plan(n, p, oblur.RECT, h) as plan:
        w = plan.apply_At(torch.as_tensor(y, dtype=torch.float32).cuda()).double().cpu().numpy()
    with np.errstate(invalid="ignore", over="ignore"):
        ref = oblur.blurT_direct(y, h, oblur.RECT)
    touched = np.zeros(ref.shape, bool)
    for r, c in ((5, 60), (66, 3)):
        touched[r:r + p, c:c + p] = True
    assert np.isfinite(w[~touched]).all()
    assert (np.abs(w - ref)[~touched] <= (2 * (p + 1) + 12) * 2.0 ** -24 * ref[~touched] + 1e-14).all()
    if np.isfinite(value):
        assert np.allclose(w[touched], ref[touched], rtol=1e-5)
    elif np.isnan(value):
        assert np.isnan(w[touched]).all()
    else:
        assert (w[touched] == value).all()
