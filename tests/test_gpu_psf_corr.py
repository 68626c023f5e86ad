"""The PSF correlations of the reverse sweep on the matrix cores
(csrc/psfgrad.hip) where their blocks of 16 x 16 lags change (p = 15, 17, 33,
49: one, four, nine and sixteen blocks) and on ragged 32 x 64 tiles, against
the FP64 oracle's gradient.

Without a threshold the unrolled map is linear in the images: two steps apply
six operators each way, each within the 1e-5 of a single operator's bar.
"""
import numpy as np
import pytest

from oracle import adjoint as oadj
from paper_1504_07234_amd import mlba
from tests._util import announce, cuda, host, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes,p", [((34,), 1), ((40, 66), 9), ((66,), 15), ((64, 34), 17), ((70,), 31), ((68,), 33),
                                     ((98,), 49)])
def test_psf_gradient(sizes, p):
    announce(f"psf gradient {sizes} p={p}")
    g = np.random.Generator(np.random.PCG64(p))
    h = g.uniform(0.0, 1.0, (p, p))
    h /= h.sum()
    ys = [g.uniform(0.0, 1.0, (n, n)) for n in sizes]
    dfs = [g.standard_normal((n + p - 1, n + p - 1)) for n in sizes]
    with mlba.Unrolled(list(sizes), p, 1, cuda(h), 2, 2) as u:
        gs = [cuda(y) for y in ys]
        _, ck = u.forward(gs, alpha=0.3, mu=0.0, delta=0.5)
        got = u.backward(gs, [cuda(d) for d in dfs], ck, alpha=0.3, mu=0.0, delta=0.5)
        dpsf, dg, dal = host(got["psf"]), [host(x) for x in got["g"]], float(got["alpha"])
    refs = [oadj.unrolled_grad(y, h, 0.3, np.zeros(9), 0.5, 2, 1, d) for y, d in zip(ys, dfs)]
    assert rel_err(dpsf, sum(r["psf"] for r in refs)) <= 12e-5
    assert abs(dal - sum(r["alpha"] for r in refs)) <= 12e-5 * sum(abs(r["alpha"]) for r in refs)
    for a, r in zip(dg, refs):
        assert rel_err(a, r["g"]) <= 12e-5
