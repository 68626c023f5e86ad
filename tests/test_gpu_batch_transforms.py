"""The compiled transforms in the batched kernels at the sides whose sequences
take several waves (768, 1024: two sequences to a workgroup of 256 threads, an
odd number of BCCB columns; 1536: one) and around them: every image of a batch
equals its own plan's restoration bit for bit, and the gradient, whose spectral
pass transforms the columns once more, the FP64 oracle's.

Without a threshold the unrolled map is linear in the images: one step applies
three operators each way, each within the 1e-5 of a single operator's bar.
"""
import numpy as np
import pytest
import torch

from oracle import adjoint as oadj
from paper_1504_07234_amd import mlba
from tests._util import announce, cuda, host, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", [mlba.BCCB, mlba.DCT])
@pytest.mark.parametrize("sides", [[384, 512], [768], [1024], [1536], [64, 768, 1024, 96]])
def test_batch_equals_plans(sides, kind):
    announce(f"batched transforms {sides} kind={kind}")
    g = np.random.Generator(np.random.PCG64(sum(sides)))
    h = g.uniform(0.1, 1.0, (5, 5))
    psf = torch.as_tensor((h / h.sum()).astype(np.float32)).cuda()
    plans = [mlba.Plan(n, 5, mlba.RECT, kind, 1, psf) for n in sides]
    ys = [torch.as_tensor(g.uniform(0.0, 1.0, (n, n)).astype(np.float32)).cuda() for n in sides]
    one = [p.restore(y, alpha=0.05, mu=1e-3, delta=0.3, iters=2)[0].clone() for p, y in zip(plans, ys)]
    with mlba.Batch(plans, max_iters=2) as batch:
        many, _ = batch.restore(ys, alpha=0.05, mu=1e-3, delta=0.3, iters=2)
        torch.cuda.synchronize()
        for a, b in zip(one, many):
            assert torch.equal(a, b)
    for p in plans:
        p.close()


@pytest.mark.parametrize("n", [512, 768, 1024, 1536])
def test_gradient(n):
    announce(f"batched gradient n={n}")
    p = 3
    g = np.random.Generator(np.random.PCG64(n))
    h = g.uniform(0.1, 1.0, (p, p))
    h /= h.sum()
    y = g.uniform(0.0, 1.0, (n, n))
    df = g.uniform(0.5, 1.5, (n + p - 1, n + p - 1))  # no cancellation in the sums
    with mlba.Unrolled([n], p, 1, cuda(h), 1, 1) as u:
        _, ck = u.forward([cuda(y)], alpha=0.3, mu=0.0, delta=0.5)
        got = u.backward([cuda(y)], [cuda(df)], ck, alpha=0.3, mu=0.0, delta=0.5)
        dpsf, dg, dal = host(got["psf"]), host(got["g"][0]), float(got["alpha"])
    ref = oadj.unrolled_grad(y, h, 0.3, np.zeros(9), 0.5, 1, 1, df)
    assert rel_err(dg, ref["g"]) <= 6e-5
    assert rel_err(dpsf, ref["psf"]) <= 6e-5
    assert abs(dal - ref["alpha"]) <= 6e-5 * abs(ref["alpha"])
