"""The compiled short transforms of the preconditioner (csrc/fft_seq.hpp; sides
2^a and 3 2^a from 64 to 1536) and their neighbours on the run-time plan, P
against the FP64 oracle.

Tolerance: two transforms along two axes, at most log2(1536) < 11 butterfly
levels each, one rounding (2^-24) of the running value per level in the 2-norm;
alpha = 1 keeps the filter from amplifying it.
"""
import numpy as np
import pytest
import torch

from oracle import alg2 as oa2
from oracle import precond as opc
from paper_1504_07234_amd import mlba

pytestmark = pytest.mark.gpu

TOL = 2 * 2 * 11 * 2.0 ** -24


@pytest.mark.parametrize("kind", [mlba.BCCB, mlba.DCT])
@pytest.mark.parametrize("n", [48, 64, 66, 96, 128, 130, 192, 256, 384, 512, 514, 768, 1024, 1280, 1536, 1600])
def test_apply_p(n, kind):
    g = np.random.Generator(np.random.PCG64(n))
    h = g.uniform(0.0, 1.0, (9, 9))
    h = (h / h.sum()).astype(np.float32)
    r = g.standard_normal((n, n)).astype(np.float32)
    with mlba.Plan(n, 9, mlba.RECT, kind, 2, torch.as_tensor(h).cuda()) as plan:
        t = plan.apply_P(torch.as_tensor(r).cuda(), 1.0).double().cpu().numpy()
    ref = opc.apply(r.astype(np.float64), h.astype(np.float64), 1.0, kind)
    assert np.linalg.norm(t - ref) <= TOL * np.linalg.norm(ref)


# Bluestein form over m = 64 .. 2048: per axis four m-point transforms of at
# most 11 levels and six products; the spectrum of the chirp is flat to within a
# factor of 2.
BLUE_TOL = 2 * 2 * (4 * 11 + 6) * 2.0 ** -24


@pytest.mark.parametrize("kind", [mlba.BCCB, mlba.DCT])
@pytest.mark.parametrize("n", [14, 22, 34, 62, 66, 126, 130, 226, 254, 258, 510, 514, 1022])
def test_apply_p_bluestein(n, kind):
    g = np.random.Generator(np.random.PCG64(n))
    h = g.uniform(0.0, 1.0, (5, 5))
    h = (h / h.sum()).astype(np.float32)
    r = g.standard_normal((n, n)).astype(np.float32)
    with mlba.Plan(n, 5, mlba.RECT, kind, 1, torch.as_tensor(h).cuda()) as plan:
        t = plan.apply_P(torch.as_tensor(r).cuda(), 1.0).double().cpu().numpy()
    ref = opc.apply(r.astype(np.float64), h.astype(np.float64), 1.0, kind)
    assert np.linalg.norm(t - ref) <= BLUE_TOL * np.linalg.norm(ref)


@pytest.mark.parametrize("n,kind", [(64, mlba.BCCB), (96, mlba.DCT), (256, mlba.BCCB), (768, mlba.DCT)])
def test_norms_from_the_column_pass(n, kind):
    """||r^k|| summed inside P's column pass equals the separate sum's, which a
    run with a discrepancy stop takes."""
    g = np.random.Generator(np.random.PCG64(n + 1))
    h = g.uniform(0.0, 1.0, (7, 7))
    psf = torch.as_tensor((h / h.sum()).astype(np.float32)).cuda()
    y = torch.as_tensor(g.uniform(0.0, 1.0, (n, n)).astype(np.float32)).cuda()
    with mlba.Plan(n, 7, mlba.RECT, kind, 2, psf) as plan:
        f1, a = plan.restore(y, alpha=0.1, delta=0.2, iters=6, implicit=True)
        f2, b = plan.restore(y, alpha=0.1, delta=0.2, iters=6, implicit=True, stop=(0.0, 1.0, 1))
    assert torch.equal(f1, f2)
    assert np.allclose(a.rnorm, b.rnorm, rtol=1e-13)


@pytest.mark.parametrize("n", [48, 64, 512, 514, 1000, 1024])
def test_algorithm2_vectors(n):
    """The PCG's vector updates inside P's row passes and in the sum of q . d: run-time,
    compiled and Bluestein plans; n^2 below, at and above one element per thread.
    Same steps and the bound of the other comparisons with the oracle, 1e-4."""
    g = np.random.Generator(np.random.PCG64(n + 2))
    h = g.uniform(0.5, 1.0, (5, 5))
    h = (h / h.sum()).astype(np.float32)
    y = g.uniform(0.0, 1.0, (n, n)).astype(np.float32)
    iters, steps = 2, 3
    ref = oa2.alg2(y.astype(np.float64), h.astype(np.float64), mlba.RECT, mlba.BCCB, 1, np.full(iters, 0.1),
                   np.full(iters + 1, 0.8), 1e-3, iters, beta_max=steps, tol=1e-12)
    with mlba.Plan(n, 5, mlba.RECT, mlba.BCCB, 1, torch.as_tensor(h).cuda()) as plan:
        f, info = plan.restore(torch.as_tensor(y).cuda(), alpha=0.1, mu=1e-3, delta=0.8, iters=iters,
                               method=mlba.ALG2, pcg=(steps, 1e-12))
        f = f.double().cpu().numpy()
    assert info.pcg_steps == ref["betas"].tolist()
    assert np.linalg.norm(f - ref["f"]) <= 1e-4 * np.linalg.norm(ref["f"])
