"""The split of the matrix-core blur (csrc/conv.hip) where its three bfloat16 parts
cannot hold a float32 value: windows and PSFs so small that the third part leaves
bfloat16's range, and PSFs beyond its largest value or not finite.

Tolerance: with nonnegative data the plain tap loop rounds once (2^-24) per tap, the
matrix form at most 2 (p + 1) + 12 times; a product below float32's normal range
is rounded to 2^-149.
"""
import numpy as np
import pytest
import torch

from oracle import blur as oblur
from paper_1504_07234_amd import mlba
from tests._util import announce

pytestmark = pytest.mark.gpu


def _plan(n, p, bc, h):
    return mlba.Plan(n, p, bc, mlba.NONE, 1, torch.as_tensor(h, dtype=torch.float32).cuda())


def _data(n, p, seed):
    g = np.random.Generator(np.random.PCG64(seed))
    h = g.uniform(0.2, 1.0, (p, p)).astype(np.float32).astype(np.float64)
    y = g.uniform(0.2, 1.0, (n, n)).astype(np.float32).astype(np.float64)
    return h, y


def _check(h, y, bc, w, p):
    ref = oblur.blurT_direct(y, h, bc)
    roundings = max(p * p, 2 * (p + 1) + 12) + 4  # folds add at most four values
    tol = roundings * 2.0 ** -24 * np.abs(ref) + (p * p + 4) * 2.0 ** -149
    most = float(np.finfo(np.float32).max)
    assert np.isposinf(w[ref - tol > most]).all()  # beyond float32
    near = (ref + tol >= most) & (ref - tol <= most)
    fits = ref + tol < most
    assert (np.abs(w - ref)[fits] <= tol[fits]).all()
    assert (np.isposinf(w[near]) | (w[near] > 0.999 * most)).all()


@pytest.mark.parametrize("p", [5, 27])
@pytest.mark.parametrize("bc", [oblur.RECT, oblur.REFLECT, oblur.PERIODIC, oblur.ZERO])
@pytest.mark.parametrize("ey,eh", [(-40, 0), (-94, 0), (-96, 0), (-110, 0), (-118, 0), (-122, 0), (30, -118), (0, -122),
                                   (-50, -50), (100, 20)])
def test_scale(p, bc, ey, eh):
    announce(f"conv split scale 2^{ey} 2^{eh} p={p} bc={bc}")
    n = 70
    h, y = _data(n, p, 10 * p + bc)
    h, y = h * 2.0 ** eh, y * 2.0 ** ey
    with _plan(n, p, bc, h) as plan:
        w = plan.apply_At(torch.as_tensor(y, dtype=torch.float32).cuda()).double().cpu().numpy()
    _check(h, y, bc, w, p)


def test_small_tile_beside_large():
    """Tiles of tiny values next to tiles of ordinary ones: each is as accurate as alone."""
    n, p = 200, 5
    h, y = _data(n, p, 3)
    y[:, 100:] *= 2.0 ** -118
    with _plan(n, p, oblur.RECT, h) as plan:
        w = plan.apply_At(torch.as_tensor(y, dtype=torch.float32).cuda()).double().cpu().numpy()
    ref = oblur.blurT_direct(y, h, oblur.RECT)
    right = slice(192, None)  # these tiles see tiny values only
    assert (np.abs(w - ref)[:, right] <= (p * p + 4) * 2.0 ** -24 * ref[:, right]).all()
    left = slice(0, 64)
    assert (np.abs(w - ref)[:, left] <= (p * p + 4) * 2.0 ** -24 * ref[:, left]).all()


@pytest.mark.parametrize("p", [5, 27])
def test_largest_tap(p):
    """A finite tap beyond bfloat16's largest value, 3.3895e38."""
    n = 40
    h, y = _data(n, p, p)
    h[1, 2] = np.float64(np.float32(3.4e38))
    y *= 0.25
    with _plan(n, p, oblur.RECT, h) as plan:
        w = plan.apply_At(torch.as_tensor(y, dtype=torch.float32).cuda()).double().cpu().numpy()
    _check(h, y, oblur.RECT, w, p)


@pytest.mark.parametrize("p", [5, 27])
@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan])
def test_tap_not_finite(p, value):
    """Every output touches every tap: the tap's infinity where a positive value lies
    under it, NaN where a zero of the extension does."""
    n = 40
    h, y = _data(n, p, p + 1)
    h[2, 1] = value
    with _plan(n, p, oblur.RECT, h) as plan:
        w = plan.apply_At(torch.as_tensor(y, dtype=torch.float32).cuda()).cpu().numpy()
    inside = oblur.blurT_direct(np.ones((n, n)), np.where(np.arange(p * p).reshape(p, p) == 2 * p + 1, 1.0, 0.0),
                                oblur.RECT) > 0.5
    assert np.isnan(w[~inside]).all()
    if np.isnan(value):
        assert np.isnan(w).all()
    else:
        assert (w[inside] == value).all()
