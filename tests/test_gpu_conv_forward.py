"""The direct blur on the matrix cores inside an iteration with the implicit state:
the forward product g - A u with its norm and the accumulating A^T, which no
single operator reaches.  P = I, one level, no threshold, step 1: the kernels of the
synthesis then give u = omega exactly for small integers and for constants.

Tolerances.  Exact cases: every product and sum fits float32, so the results are
the integers themselves.  Otherwise a sum takes at most K = 2 (p + 1) + 12
roundings of 2^-24 of its size (nonnegative data), in the 2-norm sqrt(K) of them.
"""
import numpy as np
import pytest
import torch

from oracle import blur as oblur
from paper_1504_07234_amd import mlba
from tests._util import announce

pytestmark = pytest.mark.gpu

SIZES = [(15, 3), (16, 9), (17, 1), (40, 5), (63, 17), (64, 25), (65, 25), (49, 27), (64, 31), (70, 7), (127, 33),
         (130, 49)]
BCS = [oblur.RECT, oblur.REFLECT, oblur.PERIODIC, oblur.ZERO, oblur.ANTIREFLECT]


def _cu(x):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=torch.float32).cuda()


def _step(n, p, bc, h, g, omega):
    """(omega + A^T (g - A omega), ||g - A omega||) of one iteration."""
    with mlba.Plan(n, p, bc, mlba.NONE, 1, _cu(h)) as plan:
        z = _cu(omega)
        _, info = plan.restore(_cu(g), mu=0.0, delta=1.0, iters=1, z=z, implicit=True)
        return z.double().cpu().numpy(), info.rnorm[0]


def _integers(n, p, bc, seed, most):
    g = np.random.Generator(np.random.PCG64(seed))
    N = n + p - 1 if bc == oblur.RECT else n
    return (g.integers(0, most, (N, N)).astype(np.float64), g.integers(0, most, (n, n)).astype(np.float64), g)


@pytest.mark.parametrize("bc", BCS)
@pytest.mark.parametrize("n,p", SIZES)
def test_one_tap(n, p, bc):
    """PSFs of one tap, in a corner, at an edge, in the centre and anywhere: shifts, exactly."""
    announce(f"one tap n={n} p={p} bc={bc}")
    omega, g, rng = _integers(n, p, bc, 100 * n + p + bc, 16)
    c = (p - 1) // 2
    spots = {(0, 0), (0, p - 1), (p - 1, 0), (p - 1, p - 1), (c, c), (0, c), tuple(rng.integers(0, p, 2).tolist())}
    for a, b in sorted(spots):
        h = np.zeros((p, p))
        h[a, b] = 1.0
        z, rn = _step(n, p, bc, h, g, omega)
        r = g - oblur.blur_direct(omega, h, bc)
        assert np.array_equal(z, omega + oblur.blurT(r, h, bc, "direct")), (a, b)
        assert abs(rn - np.linalg.norm(r)) <= 1e-14 * np.linalg.norm(r), (a, b)


@pytest.mark.parametrize("bc", BCS)
@pytest.mark.parametrize("n,p", [(63, 17), (64, 31), (130, 49), (520, 15), (900, 9)])
def test_streak(n, p, bc):
    """A streak of integer taps (a moved camera): few nonzero taps in every row, exactly."""
    announce(f"streak n={n} p={p} bc={bc}")
    omega, g, rng = _integers(n, p, bc, n + p + bc, 8)
    h = np.zeros((p, p))
    for i in range(p):
        h[i, (2 * i) % p] = 1.0 + i % 3
        if i % 4 == 0:
            h[p - 1 - i, i] = 2.0
    z, rn = _step(n, p, bc, h, g, omega)
    r = g - oblur.blur_direct(omega, h, bc)
    assert np.array_equal(z, omega + oblur.blurT(r, h, bc, "direct"))
    assert abs(rn - np.linalg.norm(r)) <= 1e-14 * np.linalg.norm(r)


@pytest.mark.parametrize("n,p", [(64, 1), (64, 5), (64, 9), (64, 25), (64, 27), (64, 31), (64, 49)])
def test_every_part(n, p):
    """All 24 significand bits of the taps and of the image count.  One tap: the product of two float32
    values, rounded once (the parts that are left out are below 2^-24); a lost product of the split would
    show as 2^-16 or 2^-17."""
    announce(f"split parts n={n} p={p}")
    for tap, value in ((1.00389862, 1.0), (1.0, 1.00389862), (1.00389862, 1.00389862), (0.7071068, 1.2345678)):
        h = np.zeros((p, p))
        h[p // 2, p - 1] = np.float32(tap)
        omega = np.full((n + p - 1, n + p - 1), np.float64(np.float32(value)))
        _, rn = _step(n, p, oblur.RECT, h, np.zeros((n, n)), omega)
        ref = n * h.max() * omega[0, 0]
        assert abs(rn - ref) <= (2.0 ** -25 + 2.0 ** -24 + 2.0 ** -30) * ref


@pytest.mark.parametrize("bc", BCS)
@pytest.mark.parametrize("n,p", SIZES + [(520, 15), (900, 25), (1100, 31)])
def test_dense(n, p, bc):
    """g = A omega rounded to float32: the norm of the residual is the product's error."""
    announce(f"dense n={n} p={p} bc={bc}")
    omega, _, rng = _integers(n, p, bc, 7 * n + p + bc, 1 << 10)
    h = rng.uniform(0.0, 1.0, (p, p)) ** 4 + 1e-6
    h = (h / h.sum()).astype(np.float32).astype(np.float64)
    exact = oblur.blur(omega, h, bc, "direct" if n <= 130 else "auto")
    # the pad's values reach three times the image's
    size = np.linalg.norm(exact) if bc != oblur.ANTIREFLECT else 3.0 * n * np.abs(omega).max()
    _, rn = _step(n, p, bc, h, exact.astype(np.float32), omega)
    assert rn <= (np.sqrt(2 * (p + 1) + 12) * 2.0 ** -24 + 2.0 ** -24) * size


@pytest.mark.parametrize("bc", BCS)
@pytest.mark.parametrize("n,p", [(70, 9), (70, 31)])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_not_finite(n, p, bc, value):
    """A value that is not finite in the observation reaches the pixels of omega that A^T touches from
    there, one in omega those that A^T touches from A's; the others are as without it."""
    announce(f"not finite n={n} p={p} bc={bc} {value}")
    omega, g, rng = _integers(n, p, bc, n + p + bc, 16)
    h = rng.uniform(0.5, 1.0, (p, p))
    h = (h / h.sum()).astype(np.float32).astype(np.float64)
    ones = np.ones((p, p))
    clean, _ = _step(n, p, bc, h, g, omega)

    def check(z, hit):
        """hit: the pixels touched for certain (1) or not at all (0)."""
        out = hit == 0
        assert np.isfinite(z[out]).all()
        assert (np.abs(z - clean)[out] <= 1e-5 * np.abs(clean).max()).all()
        assert not np.isfinite(z[hit == 1]).any()

    def spread(mask, forward):
        """Pixels whose pad reads a pixel of mask."""
        f = np.where(mask, np.nan, 1.0)
        with np.errstate(invalid="ignore"):
            return ~np.isfinite(oblur.blur_direct(f, ones, bc) if forward else oblur.blurT(f, ones, bc, "direct"))

    for y, x in ((5, 60), (66, 3)):
        g2 = g.copy()
        g2[y, x] = value
        mask = np.zeros((n, n), bool)
        mask[y, x] = True
        check(_step(n, p, bc, h, g2, omega)[0], spread(mask, False).astype(int))
        o2 = omega.copy()
        o2[y, x] = value
        sure, may = np.zeros(omega.shape, bool), np.zeros(omega.shape, bool)
        sure[y, x] = True
        may[max(0, y - 2):y + 3, max(0, x - 2):x + 3] = True  # W^T W reads two pixels around
        hit = np.where(spread(spread(sure, True), False), 1, np.where(spread(spread(may, True), False), 2, 0))
        hit[may] = np.where(hit[may] == 0, 2, hit[may])
        check(_step(n, p, bc, h, g, o2)[0], hit)


@pytest.mark.parametrize("p", [9, 11, 25])
@pytest.mark.parametrize("scale", [0, -90, -100, -112, -118, -122])
def test_small_values(p, scale):
    """A^T of data scaled down to where the split's third part leaves bfloat16's range: as accurate as
    unscaled (the plain loop takes p^2 roundings)."""
    announce(f"small values p={p} 2^{scale}")
    n = 96
    g = np.random.Generator(np.random.PCG64(p))
    h = g.uniform(0.2, 1.0, (p, p)).astype(np.float32).astype(np.float64)
    y = g.uniform(0.2, 1.0, (n, n)).astype(np.float32).astype(np.float64)
    with mlba.Plan(n, p, oblur.RECT, mlba.NONE, 1, _cu(h)) as plan:
        w = plan.apply_At(_cu(y * 2.0 ** scale)).double().cpu().numpy()
    ref = oblur.blurT_direct(y, h, oblur.RECT)
    assert np.linalg.norm(w * 2.0 ** -scale - ref) <= p * 2.0 ** -24 * np.linalg.norm(ref)
