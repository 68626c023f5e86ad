"""The plan autotuner keeps one choice for the calls whose direct blur runs on the
matrix cores and one for those in the order of the taps; the mode it returns, set
on another plan, gives both (a plan tuned and a plan told agree bit for bit)."""
import ctypes

import numpy as np
import pytest
import torch

from paper_1504_07234_amd import _lib, mlba
from tests._util import announce

pytestmark = pytest.mark.gpu


# 2048, p = 25: the grid lies between the two direct forms; 64, p = 9: direct for both;
# 2048, p = 31: the grid for both
@pytest.mark.parametrize("n,p", [(2048, 25), (64, 9), (2048, 31)])
def test_mode_transfers(n, p):
    announce(f"autotune transfer n={n} p={p}")
    g = np.random.Generator(np.random.PCG64(p))
    h = g.uniform(0.1, 1.0, (p, p))
    psf = torch.as_tensor((h / h.sum()).astype(np.float32)).cuda()
    y = torch.as_tensor(g.uniform(0.0, 1.0, (n, n)).astype(np.float32)).cuda()
    with mlba.Plan(n, p, mlba.RECT, mlba.BCCB, 1, psf) as a, mlba.Plan(n, p, mlba.RECT, mlba.BCCB, 1, psf) as b:
        mode = _lib.load().mlba_plan_autotune(a._h, 3, None, None)
        assert mode >= 0
        b.set_blur(mode)
        for implicit in (False, True):
            fa, fb = (q.restore(y, alpha=0.1, delta=0.3, iters=2, implicit=implicit)[0] for q in (a, b))
            assert torch.equal(fa, fb), (mode, implicit)
        assert torch.equal(a.apply_At(y), b.apply_At(y))
        u = torch.ones((a.N, a.N), device="cuda")
        assert torch.equal(a.apply_A(u), b.apply_A(u))


def test_report():
    announce("autotune report")
    h = torch.full((25, 25), 1.0 / 625, device="cuda")
    lib = _lib.load()
    with mlba.Plan(256, 25, mlba.RECT, mlba.BCCB, 1, h) as plan:
        ms = (ctypes.c_double * 2)()
        assert lib.mlba_plan_taps_ms(plan._h, ms) == 0 and list(ms) == [-1.0, -1.0]
        t = plan.autotune(reps=2)
        direct, fft, taps = sum(t["direct_ms"]), sum(t["fft_ms"]), sum(t["taps_ms"])
        assert min(t["direct_ms"] + t["fft_ms"] + t["taps_ms"]) > 0.0
        assert t["blur"] == ("fft" if fft < direct else "direct")
        assert t["blur_taps"] == "fft" or taps < fft and direct <= fft
        assert t["mode"] == {("direct", "direct"): mlba.BLUR_DIRECT, ("fft", "fft"): mlba.BLUR_FFT,
                             ("direct", "fft"): mlba.BLUR_FFT_TAPS}[(t["blur"], t["blur_taps"])]
        for mode in (-1, 3):
            with pytest.raises(_lib.MLBAError):
                plan.set_blur(mode)


def test_mode_beyond_the_grid():
    """A side whose grid would exceed 3072: refused with either mode that needs it."""
    h = torch.full((5, 5), 1.0 / 25, device="cuda")
    with mlba.Plan(3070, 5, mlba.RECT, mlba.NONE, 1, h) as plan:
        for mode in (mlba.BLUR_FFT, mlba.BLUR_FFT_TAPS):
            with pytest.raises(_lib.MLBAError):
                plan.set_blur(mode)
        assert plan.autotune(reps=1)["mode"] == mlba.BLUR_DIRECT



def _usual(plan):
    """The choice of most of three tunings (a pause of the host in one of them may turn it)."""
    return sorted(plan.autotune()["mode"] for _ in range(3))[1]


# 192, p = 31: the taps' 8-row tiles alone beat the grid (26 and 36 us), which is four times as accurate
@pytest.mark.parametrize("n,p,mode", [(64, 9, 0), (2048, 25, 2), (2048, 31, 1), (512, 17, 0), (192, 31, 2)])
def test_choice_does_not_hang_on_the_scratch(n, p, mode):
    """Forms that lie far apart (the grid takes 3, 2, 0.7, 2.6 and 1.5 times the matrix cores' time): NaN
    that an earlier restoration left in the plan's buffers does not turn the choice."""
    announce(f"autotune choice n={n} p={p}")
    h = torch.full((p, p), 1.0 / p ** 2, device="cuda")
    with mlba.Plan(n, p, mlba.RECT, mlba.BCCB, 1, h) as plan:
        assert _usual(plan) == mode
        plan.restore(torch.full((n, n), float("nan"), device="cuda"), alpha=0.1, delta=0.3, iters=2, implicit=True)
        assert _usual(plan) == mode


def test_batch_choice_does_not_hang_on_the_scratch():
    announce("batch autotune after NaN")
    h = torch.full((15, 15), 1.0 / 225, device="cuda")
    plans = [mlba.Plan(512, 15, mlba.RECT, mlba.BCCB, 1, h) for _ in range(2)]
    with mlba.Batch(plans, max_iters=2) as batch:
        batch.autotune()
        a = batch.autotune()["conv_ms"]
        batch.restore([torch.full((512, 512), float("nan"), device="cuda")] * 2, alpha=0.1, delta=0.3, iters=2,
                      implicit=True)
        b = batch.autotune()["conv_ms"]
        for x, y in zip(a, b):
            assert min(y) < 3.0 * min(x)  # the treatment of NaN takes 20 times as long
    for p in plans:
        p.close()


@pytest.mark.parametrize("implicit", [False, True])
def test_batch_tuner_leaves_the_state(implicit):
    """The tuner after a restoration with the caller's state: it reads and writes the plans' scratch, not
    the last call's buffers, and the next call carries on as without it."""
    announce(f"batch autotune after a restoration, implicit={implicit}")
    g = np.random.Generator(np.random.PCG64(5))
    h = torch.as_tensor(g.uniform(0.1, 1.0, (9, 9)).astype(np.float32) / 45).cuda()
    ys = [torch.as_tensor(g.uniform(0.0, 1.0, (n, n)).astype(np.float32)).cuda() for n in (64, 96)]
    got = []
    for tune in (False, True):
        plans = [mlba.Plan(y.shape[0], 9, mlba.RECT, mlba.BCCB, 2, h) for y in ys]
        zs = [torch.zeros((p.N, p.N) if implicit else (p.bands, p.N, p.N), device="cuda") for p in plans]
        with mlba.Batch(plans, max_iters=3) as batch:
            args = dict(alpha=0.1, mu=1e-3, delta=0.3, iters=3, implicit=implicit)
            batch.restore(ys, zs=zs, **args)
            torch.cuda.synchronize()
            before = [z.clone() for z in zs]
            if tune:
                batch.autotune(reps=2)
                assert all(torch.equal(a, b) for a, b in zip(before, zs))
            outs, _ = batch.restore(ys, zs=zs, **args)
            torch.cuda.synchronize()
            got.append([o.clone() for o in outs])
        for p in plans:
            p.close()
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("sides,kind,bc", [((64, 96, 512), mlba.BCCB, mlba.RECT), ((64, 768), mlba.DCT, mlba.REFLECT),
                                           ((65, 129), mlba.AR, mlba.ANTIREFLECT), ((80, 96), mlba.BCCB, mlba.RECT)])
def test_batch_caps(sides, kind, bc):
    """The batching caps are searched where some image's transform takes them (80 = 2^4 5)."""
    announce(f"batch caps {sides} kind={kind}")
    h = torch.full((5, 5), 1.0 / 25, device="cuda")
    plans = [mlba.Plan(n, 5, bc, kind, 1, h) for n in sides]
    with mlba.Batch(plans, max_iters=2) as batch:
        t = batch.autotune(reps=2)
    for p in plans:
        p.close()
    times = t["rows_ms"], t["cols_ms"]
    assert min(times[0] + times[1]) > 0.0
    if 80 in sides:
        assert all(len(set(x)) > 1 for x in times)
    else:
        assert (t["fft_rows_cap"], t["fft_cols_cap"]) == (0, 0) and all(len(set(x)) == 1 for x in times)
