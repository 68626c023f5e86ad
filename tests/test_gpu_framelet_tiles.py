"""Tilings of the synthesis (one wave of 64 - 2d columns, or 256 - 2d) and of the
batched analysis: the single operator against the FP64 oracle around the edges of
a tile, and batches, whose rule for the tiling looks at all images, against every
image's own plan, bit for bit.

Tolerance of the operator: per level nine masks of two passes and their sum, below
12 roundings (2^-24) of values that the masks do not enlarge in the 2-norm.
"""
import numpy as np
import pytest
import torch

from oracle import framelet as ofr
from paper_1504_07234_amd import mlba

pytestmark = pytest.mark.gpu


def _psf(p, g):
    h = g.uniform(0.1, 1.0, (p, p))
    return torch.as_tensor((h / h.sum()).astype(np.float32)).cuda()


@pytest.mark.parametrize("levels", [1, 2, 4])
@pytest.mark.parametrize("N", [24, 48, 50, 56, 58, 60, 62, 64, 66, 122, 126, 240, 242, 254, 256, 258, 602, 702])
def test_synthesis_against_oracle(N, levels):
    g = np.random.Generator(np.random.PCG64(N + levels))
    z = g.standard_normal((1 + 8 * levels, N, N)).astype(np.float32)
    with mlba.Plan(N - 2, 3, mlba.RECT, mlba.NONE, levels, _psf(3, g)) as plan:
        assert plan.N == N
        u = plan.threshold_synthesis(torch.as_tensor(z).cuda(), 0.0, 1.0).double().cpu().numpy()
    ref = ofr.synthesis(z.astype(np.float64), levels)
    assert np.linalg.norm(u - ref) <= 12 * levels * 2.0 ** -24 * np.linalg.norm(z.astype(np.float64))


@pytest.mark.parametrize("levels", [1, 4])
@pytest.mark.parametrize("sides", [[40, 46, 62], [204, 206], [256, 270, 256], [520, 64], [700, 40], [252, 776]])
def test_batch_equals_plans(sides, levels):
    """Sides on both sides of each rule, alone and mixed (204: the batch takes wide
    tiles, the plan narrow ones)."""
    g = np.random.Generator(np.random.PCG64(sum(sides)))
    plans = [mlba.Plan(n, 5, mlba.RECT, mlba.BCCB, levels, _psf(5, g)) for n in sides]
    ys = [torch.as_tensor(g.uniform(0.0, 1.0, (n, n)).astype(np.float32)).cuda() for n in sides]
    one = [p.restore(y, alpha=0.05, mu=1e-3, delta=0.3, iters=3)[0].clone() for p, y in zip(plans, ys)]
    with mlba.Batch(plans, max_iters=3) as batch:
        many, _ = batch.restore(ys, alpha=0.05, mu=1e-3, delta=0.3, iters=3)
        torch.cuda.synchronize()
        for a, b in zip(one, many):
            assert torch.equal(a, b)
    for p in plans:
        p.close()
