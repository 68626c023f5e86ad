"""The work whose speed is followed: restorations, operators and training steps as programs call them.

Every case goes through the package's public entry points.  Inputs (scene,
PSF, noise) are made from a seed on the GPU; `exact` computes the same
results in float64 with plain torch, from the definitions alone:

    x^k = delta S_mu(z^k),  r^k = g - A W^T x^k,  z^{k+1} = z^k + W A^T P_alpha r^k

A is the blur with its boundary model, W the undecimated linear B-spline
framelet, P the spectral Tikhonov preconditioner.
"""
import math

import torch

from paper_1504_07234_amd import mlba

BC = {"rect": mlba.RECT, "reflect": mlba.REFLECT, "periodic": mlba.PERIODIC, "zero": mlba.ZERO,
      "antireflect": mlba.ANTIREFLECT}
PRECOND = {"bccb": mlba.BCCB, "dct": mlba.DCT, "ar": mlba.AR}
METHOD = {"mlba": mlba.MLBA, "alg4": mlba.ALG4, "alg2": mlba.ALG2}
MU = 1e-3  # threshold of every band
DEV = "cuda"


def _restore(name, n, p, psf, bc, precond, levels, alpha, iters, implicit=True, blur="auto", method="mlba",
             step="given"):
    return {"name": name, "kind": "restore", "n": n, "p": p, "psf": psf, "bc": bc, "precond": precond,
            "levels": levels, "alpha": alpha, "iters": iters, "implicit": implicit, "blur": blur,
            "method": method, "step": step}


def listed():
    return [
        # one hand-written iteration from the single operators, at the 226 x 226 size of the paper's
        # Example 4 (31 x 31 Gaussian PSF, DCT preconditioner, 4 levels): a program with its own loop
        {"name": "operators-226", "kind": "operators", "n": 226, "p": 31, "psf": "gauss", "bc": "reflect",
         "precond": "dct", "levels": 4, "alpha": 0.02},
        # a thumbnail or a region of interest, default plan, default (explicit) state: launches count
        _restore("restore-64-rect", 64, 9, "gauss", "rect", "bccb", 1, 0.05, 50, implicit=False, blur="direct"),
        # the 196 x 196 field of view of Example 3, no 2/3/5-smooth length, antireflective, 4 levels
        _restore("restore-196-ar", 196, 31, "motion", "antireflect", "ar", 4, 0.022, 40),
        # the call of the README: tuned plan, omega state, automatic step, an out-of-focus 512 x 512 photograph
        _restore("restore-512-rect-auto", 512, 17, "disk", "rect", "bccb", 2, 0.05, 100, step="automatic"),
        # a moved camera, with imposed reflective boundary and the DCT
        _restore("restore-512-reflect-dct", 512, 17, "motion", "reflect", "dct", 2, 0.05, 50),
        # the benchmark's out-of-focus 2048 x 2048 image
        _restore("restore-2048-rect", 2048, 31, "disk", "rect", "bccb", 3, 0.02, 20),
        # the same with the frame coefficients as state, which the program keeps to resume from
        _restore("restore-2048-explicit", 2048, 31, "disk", "rect", "bccb", 3, 0.02, 10, implicit=False),
        # the antireflective model at throughput size
        _restore("restore-1025-ar", 1025, 31, "gauss", "antireflect", "ar", 3, 0.01, 30),
        # Algorithm 2: conjugate gradients on A A^T + alpha I in every iteration
        _restore("alg2-1024-rect", 1024, 15, "gauss", "rect", "bccb", 3, 0.02, 10, method="alg2"),
        # Algorithm 4 on a reflective model, direction from the DCT alone
        _restore("alg4-1536-reflect", 1536, 25, "gauss", "reflect", "dct", 4, 0.1, 20, method="alg4"),
        # a queue of uneven images restored together, replayed from one graph
        {"name": "batch-32-uneven", "kind": "batch", "count": 32, "shapes": 4, "smallest": 128, "largest": 1024,
         "levels": 2, "iters": 40, "implicit": True},
        # one training step of the unrolled network: forward, loss, gradients of every parameter
        {"name": "train-16x256", "kind": "train", "count": 16, "n": 256, "p": 15, "psf": "gauss", "levels": 2,
         "alpha": 0.05, "iters": 30, "ckpt": 5},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _smooth(n):
    for q in (2, 3, 5):
        while n % q == 0:
            n //= q
    return n == 1


def _length(rng, precond, lo, hi):
    """A side in [lo, hi] that the preconditioner's transform takes."""
    while True:
        n = _log_int(rng, lo, hi)
        if precond == "ar":
            if _smooth(2 * (n - 1)) or 2 * (n - 1) <= 1024:
                return n
        elif n % 2 == 0 and (n <= 1024 or _smooth(n)):
            return n


def _side(rng, n):
    return min(2 * rng.randrange(1, 16) + 1, n if n % 2 else n - 1)


def draw(rng):
    """Sides 32 to 2048 (odd, ragged and unsmooth ones among them), PSF sides 3 to 31, every boundary
    model with the preconditioners it pairs with, 1 to 4 levels, both states, the three methods, batches
    and training steps."""
    what = rng.choice(("operators", "restore", "restore", "restore", "restore", "batch", "train"))
    alpha = round(math.exp(rng.uniform(math.log(0.01), math.log(0.2))), 4)
    shape = rng.choice(("gauss", "gauss", "motion", "disk"))
    if what == "batch":
        implicit = rng.random() < 0.6
        return {"kind": "batch", "count": rng.randrange(6, 25), "shapes": rng.randrange(1 << 20),
                "smallest": rng.choice((48, 96, 128)), "largest": rng.choice((256, 512, 1024)),
                "levels": rng.randrange(1, 4), "iters": rng.randrange(5, 31 if implicit else 13),
                "implicit": implicit}
    if what == "train":
        n = 2 * _log_int(rng, 20, 128)
        return {"kind": "train", "count": rng.randrange(2, 17), "n": n, "p": 2 * rng.randrange(2, 9) + 1,
                "psf": shape, "levels": rng.randrange(1, 4), "alpha": max(alpha, 0.02),
                "iters": rng.randrange(6, 31), "ckpt": rng.randrange(2, 7)}
    bc, precond = rng.choice((("rect", "bccb"), ("rect", "bccb"), ("rect", "dct"), ("reflect", "dct"),
                              ("reflect", "bccb"), ("periodic", "bccb"), ("zero", "bccb"), ("antireflect", "ar"),
                              ("antireflect", "dct")))
    n = _length(rng, precond, 32, 2048)
    levels = rng.randrange(1, 5)
    p = _side(rng, n)
    if what == "operators":
        return {"kind": "operators", "n": n, "p": p, "psf": shape, "bc": bc, "precond": precond,
                "levels": levels, "alpha": alpha}
    method = rng.choice(("mlba", "mlba", "mlba", "alg2", "alg4"))
    if method == "alg4" and (bc == "rect" or shape == "motion") or method == "alg2" and bc == "antireflect":
        method = "mlba"
    if method == "alg4":
        alpha = max(alpha, 0.05)
    most = max(4, min(15 if method == "alg2" else 50, int(40 * (1024 / n) ** 2)))
    c = _restore("", n, p, shape, bc, precond, levels, alpha, rng.randrange(2, most) + 2,
                 implicit=rng.random() < 0.6, blur=rng.choice(("auto", "auto", "direct")), method=method)
    del c["name"]
    return c


# ---- inputs --------------------------------------------------------------

def _psf(p, kind, gen):
    """p x p, nonnegative, sum 1: Gaussian, out-of-focus disk, or a motion streak of random direction."""
    c = (p - 1) // 2
    y, x = torch.meshgrid(torch.arange(p, dtype=torch.float64) - c, torch.arange(p, dtype=torch.float64) - c,
                          indexing="ij")
    if kind == "gauss":
        h = torch.exp(-(x * x + y * y) / (2 * max(0.6, p / 8.0) ** 2))
    elif kind == "disk":
        h = (x * x + y * y <= c * c + 0.25).double()
    else:
        th = math.pi * float(torch.rand((), generator=gen, dtype=torch.float64))
        along, across = x * math.cos(th) + y * math.sin(th), y * math.cos(th) - x * math.sin(th)
        h = torch.clamp(1.0 - across.abs(), min=0.0) * (along.abs() <= 0.45 * p)
    return (h / h.sum()).to(DEV)


def _scene(m, gen):
    """Painted rectangles and disks plus smooth waves, in [0, 1], m x m float64."""
    t = torch.arange(m, device=DEV, dtype=torch.float32)
    v = torch.rand(18, 5, generator=gen, dtype=torch.float64).tolist()
    img = torch.zeros(m, m, device=DEV)
    for i, (a, b, c, d, e) in enumerate(v):
        if i < 12:
            h, w = m * (1 / 16 + a * 13 / 48), m * (1 / 16 + b * 13 / 48)
            y0, x0 = int(c * m - h / 2), int(d * m - w / 2)
            img[max(0, y0):max(0, int(y0 + h)), max(0, x0):max(0, int(x0 + w))] = e
        else:
            r = m * (1 / 32 + a * 3 / 32)
            img = torch.where((t[:, None] - b * m) ** 2 + (t[None, :] - c * m) ** 2 <= r * r, e, img)
    wave = torch.sin(0.11 * t[:, None] + 0.07 * t[None, :]) + torch.cos(0.23 * t[None, :] - 0.05 * t[:, None])
    img = (img + 0.05 * wave).double()
    return (img - img.min()) / (img.max() - img.min())


def _observe(n, p, kind, seed, noise=0.01):
    """(g, psf, scene): the valid part of a blurred (n + p - 1)^2 scene plus white noise, float32."""
    gen = torch.Generator().manual_seed(seed)
    h = _psf(p, kind, gen).float().double()
    scene = _scene(n + p - 1, gen)
    b = _conv_valid(scene, h)
    dev = torch.Generator(device=DEV).manual_seed(seed)
    xi = torch.randn(n, n, generator=dev, device=DEV, dtype=torch.float64)
    g = b + noise * torch.linalg.vector_norm(b) / torch.linalg.vector_norm(xi) * xi
    return g.float(), h.float(), scene.float()


def _batch_shapes(case):
    """(n, p, sigma-free PSF kind, alpha) of each image, from the case's own shape number."""
    gen = torch.Generator().manual_seed(case["shapes"])
    sides = [s for s in (48, 64, 96, 128, 192, 256, 384, 512, 768, 1024) if case["smallest"] <= s <= case["largest"]]
    got = []
    for _ in range(case["count"]):
        i, j = torch.randint(0, 1 << 20, (2,), generator=gen).tolist()
        got.append((sides[i % len(sides)], 2 * (j % 9) + 9,
                    round(0.02 + 0.18 * float(torch.rand((), generator=gen)), 4)))
    return got


def _step(model, alpha):
    """A step that satisfies delta ||A^T P_alpha A|| < 1 (power iteration in float64)."""
    gen = torch.Generator(device=DEV).manual_seed(7)
    v = torch.randn(model.N, model.N, generator=gen, device=DEV, dtype=torch.float64)
    for _ in range(12):
        v = model.At(model.P(model.A(v / torch.linalg.vector_norm(v)), alpha))
    return round(0.8 / max(float(torch.linalg.vector_norm(v)), 0.8), 6)


def _one(case, seed):
    """Inputs of a single-image case and its step."""
    g, h, scene = _observe(case["n"], case["p"], case["psf"], seed)
    model = _Model(h.double(), case["n"], case["bc"], case["precond"], case["levels"])
    delta = 1.0 if case.get("method") == "alg4" else _step(model, case["alpha"])
    return g, h, scene, model, delta


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("restore", "operators"):
        g, h, scene, _, delta = _one(case, seed)
        plan = mlba.Plan(case["n"], case["p"], BC[case["bc"]], PRECOND[case["precond"]], case["levels"], h)
        st = {"case": case, "plan": plan, "g": g, "delta": delta}
        if kind == "operators":
            st["z"] = plan.analysis(_start_image(case, scene))
            st["u"], st["w"] = plan._new(plan.N, plan.N), plan._new(plan.N, plan.N)
            st["r"], st["t"] = plan._new(plan.n, plan.n), plan._new(plan.n, plan.n)
            st["next"] = torch.empty_like(st["z"])
            return st
        if case["blur"] == "auto":
            plan.autotune()
        if not case["implicit"]:
            st["z"] = plan._new(plan.bands, plan.N, plan.N)
        return st
    if kind == "batch":
        st = {"case": case, "g": [], "plans": [], "alpha": [], "delta": []}
        for i, (n, p, alpha) in enumerate(_batch_shapes(case)):
            g, h, _ = _observe(n, p, "gauss", seed * 1000 + i)
            st["g"].append(g)
            st["alpha"].append(alpha)
            st["delta"].append(_step(_Model(h.double(), n, "rect", "bccb", case["levels"]), alpha))
            st["plans"].append(mlba.Plan(n, p, mlba.RECT, mlba.BCCB, case["levels"], h))
        st["batch"] = mlba.Batch(st["plans"], case["iters"])
        st["batch"].autotune()
        st["out"] = [p._new(p.N, p.N) for p in st["plans"]]
        return st
    g, h, truth, delta = _train_inputs(case, seed)
    engine = mlba.Unrolled([case["n"]] * case["count"], case["p"], case["levels"], h, case["iters"], case["ckpt"])
    mu = torch.full((engine.bands,), MU, device=DEV)
    return {"case": case, "engine": engine, "truth": truth, "delta": delta,
            "params": [t.requires_grad_() for t in (g, h, torch.tensor(case["alpha"], device=DEV), mu)]}


def _start_image(case, scene):
    """The image whose coefficients an operators case starts from: the scene, cropped to the unknown."""
    c = 0 if case["bc"] == "rect" else (case["p"] - 1) // 2
    side = scene.shape[0] - 2 * c
    return scene[c:c + side, c:c + side].contiguous()


def _train_inputs(case, seed):
    gs, truths = [], []
    for i in range(case["count"]):
        g, h, truth = _observe(case["n"], case["p"], case["psf"], seed * 1000 + i)
        gs.append(g)
        truths.append(truth)
    h = _observe(8, case["p"], case["psf"], seed)[1]
    model = _Model(h.double(), case["n"], "rect", "bccb", case["levels"])
    return torch.stack(gs), h, torch.stack(truths), _step(model, case["alpha"])


# ---- one pass ------------------------------------------------------------

def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "restore":
        z = st.get("z")
        if z is not None:
            z.zero_()
        f, info = st["plan"].restore(st["g"], alpha=case["alpha"], mu=MU,
                                     delta=0.0 if case["step"] == "automatic" else st["delta"],
                                     iters=case["iters"], z=z, implicit=case["implicit"],
                                     method=METHOD[case["method"]])
        out = {"f": f, "rnorm": torch.tensor(info.rnorm)}
        if z is not None:
            out["z"] = z
        return out
    if kind == "operators":
        plan = st["plan"]
        z = st["next"].copy_(st["z"])
        plan.threshold_synthesis(z, MU, st["delta"], out=st["u"])
        plan.residual(st["g"], st["u"], out=st["r"])
        plan.apply_P(st["r"], case["alpha"], out=st["t"])
        plan.apply_At(st["t"], out=st["w"])
        plan.analysis_update(st["w"], z)
        return {"u": st["u"], "r": st["r"], "t": st["t"], "w": st["w"], "z": z}
    if kind == "batch":
        outs, _ = st["batch"].restore(st["g"], alpha=st["alpha"], mu=MU, delta=st["delta"], iters=case["iters"],
                                      outs=st["out"], implicit=case["implicit"])
        return outs
    g, h, alpha, mu = st["params"]
    f = mlba.unrolled_mlba(g, h, alpha, mu, st["engine"], st["delta"])
    loss = ((f - st["truth"]) ** 2).sum()
    grads = torch.autograd.grad(loss, st["params"])
    return {"f": f.detach(), "dg": grads[0], "dpsf": grads[1], "dalpha": grads[2], "dmu": grads[3]}


# ---- what a pass cannot do without ------------------------------------------

def _flops_iteration(n, p, N, levels, method="mlba"):
    """Threshold, synthesis (and analysis) of the frame; two blurs, by taps or transforms; P."""
    m = n + p - 1
    blur = min(2.0 * p * p * n * n, 10.0 * m * m * math.log2(m))
    pre = 10.0 * n * n * math.log2(n)
    times = {"mlba": (2, 1), "alg4": (1, 1), "alg2": (2 + 2 * 5, 6)}[method]
    return 119.0 * levels * N * N + times[0] * blur + times[1] * pre


def work(case):
    """Flops of the iterations; bytes: per iteration the state read and written once and g read once,
    then the results written once."""
    kind = case["kind"]
    if kind in ("restore", "operators"):
        n, p = case["n"], case["p"]
        N = n + p - 1 if case["bc"] == "rect" else n
        planes = 1 if case.get("implicit") else 8 * case["levels"] + 1
        iters = case.get("iters", 1)
        extra = 4.0 * (N * N + n * n) if kind == "operators" else 0.0  # u and w, r and t come back as well
        return {"flops": iters * _flops_iteration(n, p, N, case["levels"], case.get("method", "mlba")),
                "bytes": iters * (8.0 * planes * N * N + 4.0 * n * n) + 4.0 * N * N + 2 * extra}
    if kind == "batch":
        w = {"flops": 0.0, "bytes": 0.0}
        planes = 1 if case["implicit"] else 8 * case["levels"] + 1
        for n, p, _ in _batch_shapes(case):
            N = n + p - 1
            w["flops"] += case["iters"] * _flops_iteration(n, p, N, case["levels"])
            w["bytes"] += case["iters"] * (8.0 * planes * N * N + 4.0 * n * n) + 4.0 * N * N
        return w
    # forward, one recomputation from the checkpoints, and a reverse sweep of about twice an iteration,
    # which also correlates two pairs of images over the PSF's support
    n, p, K = case["n"], case["p"], case["iters"]
    N = n + p - 1
    bands = 8 * case["levels"] + 1
    it = _flops_iteration(n, p, N, case["levels"])
    return {"flops": case["count"] * K * (4.0 * it + 4.0 * p * p * n * n),
            "bytes": case["count"] * (K * (4 * 8.0 * bands * N * N + 12.0 * n * n) + 8.0 * (N * N + n * n))}


# ---- the same in float64 ------------------------------------------------------

def _fast(m):
    return 1 << (m - 1).bit_length()


def _conv_valid(f, h):
    """Valid part of the 2-D convolution of the square f with h."""
    p = h.shape[0]
    M = _fast(f.shape[0])
    v = torch.fft.irfft2(torch.fft.rfft2(f, s=(M, M)) * torch.fft.rfft2(h, s=(M, M)), s=(M, M))
    return v[..., p - 1:f.shape[-1], p - 1:f.shape[-1]]


def _corr_full(y, h):
    """Full correlation: the transpose of _conv_valid."""
    m = y.shape[-1] + h.shape[0] - 1
    M = _fast(m)
    v = torch.fft.irfft2(torch.fft.rfft2(y, s=(M, M)) * torch.fft.rfft2(h.flip(0, 1), s=(M, M)), s=(M, M))
    return v[..., :m, :m]


class _Model:
    """A, A^T, P and the frame of one problem in float64."""

    def __init__(self, h, n, bc, precond, levels):
        self.h, self.n, self.bc, self.precond, self.levels = h, n, bc, precond, levels
        self.p = h.shape[0]
        self.c = (self.p - 1) // 2
        self.N = n + self.p - 1 if bc == "rect" else n
        self.bands = 8 * levels + 1
        if bc != "rect":
            self.E = self._extension()
        k = torch.arange(n, device=DEV, dtype=torch.float64)
        s = torch.arange(self.p, device=DEV, dtype=torch.float64) - self.c
        sym = (h + h.flip(0) + h.flip(1) + h.flip(0, 1)) / 4
        if precond == "bccb":
            self.lam = torch.fft.fft2(torch.roll(torch.nn.functional.pad(h, (0, n - self.p, 0, n - self.p)),
                                                 (-self.c, -self.c), (0, 1)))
        elif precond == "dct":
            cm = torch.cos(math.pi * k[:, None] * s[None, :] / n)
            self.lam = cm @ sym @ cm.T
            fwd = math.sqrt(2.0 / n) * torch.cos(math.pi * k[:, None] * (2 * k[None, :] + 1) / (2 * n))
            fwd[0] /= math.sqrt(2.0)
            self.fwd, self.inv = fwd, fwd.T
        else:
            w = math.pi * k / (n - 1)
            w[0] = w[-1] = 0.0
            cm = torch.cos(w[:, None] * s[None, :])
            self.lam = cm @ sym @ cm.T
            # columns: the two linear functions and the sines; the inverse takes the end values off first
            sine = torch.sin(math.pi * k[:, None] * k[None, :] / (n - 1))
            sine[:, 0], sine[:, -1] = 1 - k / (n - 1), k / (n - 1)
            self.inv = sine
            sines = sine[1:-1, 1:-1] * (2.0 / (n - 1))
            self.fwd = torch.zeros_like(sine)
            self.fwd[0, 0] = self.fwd[-1, -1] = 1.0
            self.fwd[1:-1, 1:-1] = sines
            self.fwd[1:-1, 0] = -(sines @ sine[1:-1, 0])
            self.fwd[1:-1, -1] = -(sines @ sine[1:-1, -1])

    def _extension(self):
        """The (n + 2c) x n matrix of the pad along one axis."""
        n, c = self.n, self.c
        E = torch.zeros(n + 2 * c, n, dtype=torch.float64)
        for r in range(n + 2 * c):
            x = r - c
            if 0 <= x < n:
                E[r, x] = 1.0
            elif self.bc == "reflect":
                E[r, -1 - x if x < 0 else 2 * n - 1 - x] = 1.0
            elif self.bc == "periodic":
                E[r, x % n] = 1.0
            elif self.bc == "antireflect":
                edge = 0 if x < 0 else n - 1
                E[r, edge] += 2.0
                E[r, 2 * edge - x] -= 1.0
        return E.to(DEV)

    def A(self, u, h=None):
        h = self.h if h is None else h
        return _conv_valid(u if self.bc == "rect" else self.E @ u @ self.E.T, h)

    def At(self, y, h=None):
        h = self.h if h is None else h
        if self.bc == "antireflect":  # the reblurring takes the transpose's place
            return self.A(y, h.flip(0, 1))
        w = _corr_full(y, h)
        return w if self.bc == "rect" else self.E.T @ w @ self.E

    def _spectral(self, r, filt):
        if self.precond == "bccb":
            return torch.fft.ifft2(torch.fft.fft2(r) * filt).real
        return self.inv @ ((self.fwd @ r @ self.fwd.T) * filt) @ self.inv.T

    def P(self, r, alpha):
        return self._spectral(r, 1.0 / (self.lam.abs() ** 2 + alpha))

    def CtP(self, r, alpha):
        return self._spectral(r, self.lam.conj() / (self.lam.abs() ** 2 + alpha) if self.precond == "bccb"
                              else self.lam / (self.lam ** 2 + alpha))

    def _taps(self, v, d, dim, odd):
        """v at x - d and x + d, extended half-sample symmetrically (odd: with the sign turned)."""
        N = v.shape[dim]
        x = torch.arange(N, device=DEV)
        got = []
        for t in (x - d, x + d):
            t = t % (2 * N)
            q = v.index_select(dim, torch.where(t < N, t, 2 * N - 1 - t))
            if odd:
                sign = torch.where(t < N, 1.0, -1.0).double()
                q = q * (sign[:, None] if dim % 2 == 0 else sign)
            got.append(q)
        return got

    def _filter(self, v, i, d, dim):
        lo, hi = self._taps(v, d, dim, False)
        return (lo + 2 * v + hi) / 4 if i == 0 else (hi - lo) * (math.sqrt(2) / 4) if i == 1 else (2 * v - lo - hi) / 4

    def _filter_t(self, v, i, d, dim):
        if i != 1:
            return self._filter(v, i, d, dim)
        lo, hi = self._taps(v, d, dim, True)
        return (lo - hi) * (math.sqrt(2) / 4)

    def W(self, v):
        got = []
        for lev in range(self.levels):
            hx = [self._filter(v, i, 2 ** lev, 1) for i in range(3)]
            got += [self._filter(hx[i], j, 2 ** lev, 0) for i in range(3) for j in range(3) if i or j]
            v = self._filter(hx[0], 0, 2 ** lev, 0)
        return torch.stack([v] + got)

    def Wt(self, z):
        v = z[0]
        for lev in reversed(range(self.levels)):
            bands = [v] + list(z[1 + 8 * lev:9 + 8 * lev])
            v = sum(self._filter_t(sum(self._filter_t(bands[3 * i + j], j, 2 ** lev, 0) for j in range(3)), i,
                                   2 ** lev, 1) for i in range(3))
        return v

    def image(self, z, delta, mu=MU):
        """W^T (delta S_mu(z))."""
        if torch.is_tensor(mu):
            mu = mu[:, None, None]
        return self.Wt(delta * torch.sign(z) * torch.clamp(z.abs() - mu, min=0.0))

    def norm(self, alpha, steps=300):
        """The largest eigenvalue of A^T P A: Lanczos with full reorthogonalisation."""
        gen = torch.Generator(device=DEV).manual_seed(3)
        q = torch.randn(self.N * self.N, generator=gen, device=DEV, dtype=torch.float64)
        Q = torch.zeros(steps, q.numel(), device=DEV, dtype=torch.float64)
        T = torch.zeros(steps, steps, dtype=torch.float64)
        Q[0] = q / torch.linalg.vector_norm(q)
        for k in range(steps):
            w = self.At(self.P(self.A(Q[k].reshape(self.N, self.N)), alpha)).reshape(-1)
            T[k, k] = float(Q[k] @ w)
            for _ in range(2):
                w = w - Q[:k + 1].T @ (Q[:k + 1] @ w)
            b = float(torch.linalg.vector_norm(w))
            if k + 1 == steps or b < 1e-12:
                return float(torch.linalg.eigvalsh(T[:k + 1, :k + 1])[-1])
            T[k, k + 1] = T[k + 1, k] = b
            Q[k + 1] = w / b

    def pcg(self, r, alpha, most=5, tol=1e-3):
        """(A A^T + alpha I)^-1 r by conjugate gradients preconditioned with P."""
        t, res = torch.zeros_like(r), r
        z = self.P(res, alpha)
        d, rho = z, float((res * z).sum())
        rho0 = rho
        for _ in range(most):
            q = self.A(self.At(d)) + alpha * d
            a = rho / float((d * q).sum())
            t, res = t + a * d, res - a * q
            z = self.P(res, alpha)
            new = float((res * z).sum())
            if math.sqrt(new / rho0) <= tol:
                break
            d, rho = z + (new / rho) * d, new
        return t


def _run64(model, g, alpha, delta, iters, method="mlba"):
    z = torch.zeros(model.bands, model.N, model.N, device=DEV, dtype=torch.float64)
    rnorm = []
    for _ in range(iters):
        r = g - model.A(model.image(z, delta))
        rnorm.append(float(torch.linalg.vector_norm(r)))
        if method == "alg4":
            w = model.CtP(r, alpha)
        else:
            w = model.At(model.P(r, alpha) if method == "mlba" else model.pcg(r, alpha))
        z += model.W(w)
    return model.image(z, delta), rnorm, z


def exact(case, seed):
    kind = case["kind"]
    if kind == "restore":
        g, _, _, model, delta = _one(case, seed)
        if case["step"] == "automatic":
            delta = 0.9 / max(model.norm(case["alpha"]), 0.9)
        f, rnorm, z = _run64(model, g.double(), case["alpha"], delta, case["iters"], case["method"])
        out = {"f": f, "rnorm": torch.tensor(rnorm)}
        if not case["implicit"]:
            out["z"] = z
        return out
    if kind == "operators":
        g, _, scene, model, delta = _one(case, seed)
        z = model.W(_start_image(case, scene).double())
        u = model.image(z, delta)
        r = g.double() - model.A(u)
        t = model.P(r, case["alpha"])
        w = model.At(t)
        return {"u": u, "r": r, "t": t, "w": w, "z": z + model.W(w)}
    if kind == "batch":
        outs = []
        for i, (n, p, alpha) in enumerate(_batch_shapes(case)):
            g, h, _ = _observe(n, p, "gauss", seed * 1000 + i)
            model = _Model(h.double(), n, "rect", "bccb", case["levels"])
            outs.append(_run64(model, g.double(), alpha, _step(model, alpha), case["iters"])[0])
        return outs
    g, h, truth, delta = _train_inputs(case, seed)
    g, truth = g.double(), truth.double()
    h = h.double().requires_grad_()
    alpha = torch.tensor(case["alpha"]).to(DEV).double().requires_grad_()
    mu = torch.full((8 * case["levels"] + 1,), MU).to(DEV).double().requires_grad_()
    fs, dgs = [], []
    total = [torch.zeros_like(t) for t in (h, alpha, mu)]
    for i in range(case["count"]):
        gi = g[i].clone().requires_grad_()
        model = _Model(h, case["n"], "rect", "bccb", case["levels"])
        z = torch.zeros(model.bands, model.N, model.N, device=DEV, dtype=torch.float64)
        for _ in range(case["iters"]):
            z = z + model.W(model.At(model.P(gi - model.A(model.image(z, delta, mu)), alpha)))
        f = model.image(z, delta, mu)
        got = torch.autograd.grad(((f - truth[i]) ** 2).sum(), (gi, h, alpha, mu))
        fs.append(f.detach())
        dgs.append(got[0])
        total = [a + b for a, b in zip(total, got[1:])]
    return {"f": torch.stack(fs), "dg": torch.stack(dgs), "dpsf": total[0], "dalpha": total[1], "dmu": total[2]}
