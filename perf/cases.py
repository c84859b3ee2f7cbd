"""Workloads of the engine over the range its users run, through the public entry points.

A case is a dict: `kind` names the entry point, the rest its sizes and options.  Inputs
are standing-wave states like those of paper_1210_5672_amd/workloads.py: a first mode of
the given amplitude and decaying random modes 2..16 drawn from the seed.  Marches run a
few steps of the step size that a march to T/4 takes (`full` steps), so a pass stays
short while every stage does the work of the full march.

kinds:
  dtn       dtn_setup of a surface and dtn_solve_multi of R columns
  dtn_dd    the same in double-double (dtn_setup_dd, dtn_solve_multi_dd)
  march     shoot_eval: r, J, dr/dT and f
  f_only    shoot_eval without the Jacobian (the driver's residual evaluations)
  adjoint   shoot_adjoint: the gradient with checkpoints
  segments  shoot_eval_segments over two meshes
  sdc       shoot_eval_sdc: r, J, dr/dT and f by SDC15 steps
  sdc_dd    shoot_eval_sdc_dd: the double-double base march
  batch     shoot_eval_batch over continuation instances of uneven size
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1210_5672_amd import workloads as W
from paper_1210_5672_amd import ww

INF = math.inf
STAGES = 12          # of the DOP853 update
SDC_EVALS = 113      # right-hand sides of an SDC15 step


def _freq(N, h, tau):
    """Largest filtered linear frequency on the grid."""
    th = lambda k: 1.0 if math.isinf(h) else math.tanh(k * h)
    return max(math.sqrt((1.0 + tau * k * k) * k * th(k)) * math.exp(-36.0 * (k / (N / 2)) ** 36)
               for k in range(1, N // 2 + 1))


def listed():
    return [
        # one DtN on the smallest problem the tests and the convergence workload use
        # (N = 64, 8 parameters): latency, launches, synchronisations
        dict(name="dtn N64 R9", kind="dtn", N=64, R=9, h=-1.0, a1=0.01, mixed=False),
        # the DtN of the largest grid with a full set of right-hand sides
        dict(name="dtn N2048 R257", kind="dtn", N=2048, R=257, h=1.0, a1=0.05, mixed=False),
        # the double-double DtN of the quadruple-precision workflow, on the headline grid
        dict(name="dtn_dd N1024 R129", kind="dtn_dd", N=1024, R=129, h=0.5, a1=0.05),
        # Jacobian marches: the mid-size validation workload (N = 256, 64 columns, 300
        # steps to T/4), then the headline one (N = 1024, 128 columns, 600 steps)
        dict(name="march N256 M64", kind="march", N=256, M=64, h=1.0, tau=0.0, a1=0.05, full=300, steps=25,
             mixed=False),
        dict(name="march N1024 M128", kind="march", N=1024, M=128, h=0.5, tau=0.02, a1=0.05, full=600, steps=24,
             mixed=False),
        # the mixed-precision form on a radix-3 grid with a ragged column count
        dict(name="march mixed N768 M137", kind="march", N=768, M=137, h=0.7, tau=0.01, a1=0.05, full=400, steps=16,
             mixed=True),
        # residual evaluations between Jacobians (most evaluations of the LM driver)
        dict(name="f_only N1024", kind="f_only", N=1024, M=128, h=0.5, tau=0.02, a1=0.05, full=600, steps=24,
             mixed=False),
        # the gradient of the adjoint minimiser (N = 512, 256 parameters, steep surface)
        dict(name="adjoint N512 M256", kind="adjoint", N=512, M=256, h=-1.0, tau=0.0, a1=0.2, full=800, steps=13,
             ckpt=5),
        # two time segments on refined meshes (768 then 1024 points, 200 columns)
        dict(name="segments N768-1024 M200", kind="segments", N=768, N2=1024, M=200, a1=0.15, rho=0.4, full=24,
             full2=144, steps=3, steps2=18),
        # SDC15 with the Jacobian (12 steps to T/4), and its double-double base march
        dict(name="sdc N512 M256", kind="sdc", N=512, M=256, h=-1.0, tau=0.0, a1=0.2, full=12, steps=2, mixed=False),
        dict(name="sdc_dd N512", kind="sdc_dd", N=512, h=-1.0, tau=0.0, a1=0.2, full=12, steps=1),
        # continuation instances of uneven size marched together
        dict(name="batch 5 instances", kind="batch", n=5, nmax=2048, pick=7, steps=5),
    ]


_SIZES = sorted(2 ** a * 3 ** b for a in range(1, 12) for b in range(7) if 16 <= 2 ** a * 3 ** b <= 2048)


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi, pow2=False):
    x = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    s = [n for n in _SIZES if lo <= n <= hi and (not pow2 or n & (n - 1) == 0)]
    return min(s, key=lambda n: abs(math.log(n / x)))


def _wave(rng):
    """Depth (-1: infinite), tension and amplitude of a continuation instance."""
    h = -1.0 if rng.random() < 0.25 else round(rng.uniform(0.1, 3.0), 4)
    tau = round(rng.uniform(0.0, 0.05), 4)
    a1 = round(rng.uniform(0.01, 0.2), 4)
    if h > 0:
        a1 = min(a1, round(0.2 * h, 4))
    return h, tau, a1


def _full(N, h, tau, cfl=4.5):
    """Steps to T/4 at the stability bound dt omega_max <= cfl (and at least 64)."""
    T = W.linear_period(INF if h < 0 else h, tau)
    return max(64, int(math.ceil(1.1 * T / 4.0 * _freq(N, INF if h < 0 else h, tau) / cfl)))


def draw(rng):
    kind = rng.choice(["dtn", "dtn", "march", "march", "march", "f_only", "adjoint", "segments", "sdc", "sdc_dd",
                       "dtn_dd", "batch"])
    h, tau, a1 = _wave(rng)
    if kind == "dtn":
        return dict(kind=kind, N=_size(rng, 16, 2048), R=_logint(rng, 1, 257), h=h, a1=a1, mixed=rng.random() < 0.4)
    if kind == "dtn_dd":
        return dict(kind=kind, N=_size(rng, 16, 1024, pow2=True), R=_logint(rng, 1, 129), h=h, a1=a1)
    if kind in ("march", "f_only"):
        N = _size(rng, 32, 1024)
        M = min(_logint(rng, 2, 200), N // 2)
        return dict(kind=kind, N=N, M=M, h=h, tau=tau, a1=a1, full=_full(N, h, tau), steps=rng.randint(3, 20),
                    mixed=rng.random() < 0.3)
    if kind == "adjoint":
        N = _size(rng, 32, 512)
        return dict(kind=kind, N=N, M=min(_logint(rng, 2, 256), N // 2), h=h, tau=tau, a1=a1, full=_full(N, h, tau),
                    steps=rng.randint(3, 13), ckpt=rng.randint(2, 6))
    if kind == "segments":
        N = _size(rng, 48, 768)
        rho = round(rng.uniform(0.4, 0.9), 3)
        N2 = min(n for n in _SIZES if n >= N * 8.0 / (5.0 + 3.0 * rho))
        return dict(kind=kind, N=N, N2=N2, M=min(_logint(rng, 4, 200), N // 2), a1=round(rng.uniform(0.01, 0.15), 4),
                    rho=rho, full=24, full2=144, steps=rng.randint(1, 3), steps2=rng.randint(3, 18))
    if kind == "sdc":
        N = _size(rng, 32, 512)
        return dict(kind=kind, N=N, M=min(_logint(rng, 2, 256), N // 2), h=h, tau=0.0, a1=a1,
                    full=max(12, _full(N, h, 0.0, 1.8)), steps=1, mixed=rng.random() < 0.3)
    if kind == "sdc_dd":
        N = _size(rng, 16, 512, pow2=True)
        return dict(kind=kind, N=N, h=h, tau=0.0, a1=a1, full=max(12, _full(N, h, 0.0, 1.8)), steps=1)
    return dict(kind="batch", n=rng.randint(2, 5), nmax=rng.choice([512, 768, 1024, 1536]),
                pick=rng.randint(0, 10 ** 6), steps=rng.randint(2, 5))


# ----- inputs -------------------------------------------------------------------------

def _depth(case):
    return INF if case.get("h", -1.0) <= 0 else float(case["h"])


def _modes(rng, a1, M):
    p = np.zeros(max(M, 1))
    p[0] = a1 * (1.0 + 0.02 * rng.normal())
    for k in range(2, min(16, M) + 1):
        p[k - 1] = rng.normal(0.0, 1e-3 * 2.0 ** (-k))
    return p


def _surface(rng, N, a1):
    a = W.grid(N)
    eta = a1 * (1.0 + 0.02 * rng.normal()) * np.cos(a)
    for k in range(2, min(12, N // 3) + 1):
        eta += 0.2 * a1 * 2.0 ** (-k) * (rng.normal() * np.cos(k * a) + rng.normal() * np.sin(k * a))
    return eta


def _instances(case):
    """The batch's instances: sizes, depths, tensions and steps drawn from `pick`."""
    rng = np.random.default_rng(1000 + int(case["pick"]))
    sizes = [n for n in (256, 384, 512, 768, 1024, 1536, 2048) if n <= case["nmax"]]
    out = []
    for i in range(case["n"]):
        N = sizes[-1] if i == 0 else int(rng.choice(sizes))
        h = -1.0 if rng.uniform() < 0.25 else float(rng.uniform(0.1, 3.0))
        tau = float(rng.uniform(0.0, 0.05))
        a1 = float(rng.uniform(0.01, 0.2))
        if h > 0:
            a1 = min(a1, 0.2 * h)
        M = min(int(rng.integers(32, 257)), N // 2)
        out.append(dict(kind="march", N=N, M=M, h=h, tau=tau, a1=a1, full=_full(N, h, tau), steps=case["steps"],
                        mixed=False))
    return out


def _period(case):
    """The T of the shortened march: `steps` steps of the full march's dt."""
    return W.linear_period(_depth(case), case["tau"]) * case["steps"] / case["full"]


def _march_host(case, seed):
    rng = np.random.default_rng([int(seed), 17])
    return _modes(rng, case["a1"], case["M"])


def _shoot_context(case, seed, stream=None):
    N, M = case["N"], case["M"]
    ctx = ww.Context(n_max=max(64, N), r_max=M + 1, mixed=bool(case.get("mixed", False)), stream=stream)
    ctx.shoot_setup(N, _depth(case), case["tau"], 1.0, ww.to_dev(W.cosine_basis(N, M)), ww.to_dev(np.zeros(2 * N)))
    return ctx, ww.to_dev(_march_host(case, seed))


def _dtn_host(case, seed):
    rng = np.random.default_rng([int(seed), 5])
    return _surface(rng, case["N"], case["a1"]), rng.standard_normal((case["N"], case["R"]))


def prepare(case, seed):
    kind = case["kind"]
    st = dict(case=case)
    if kind == "dtn":
        eta, rhs = _dtn_host(case, seed)
        st["ctx"] = ww.Context(n_max=max(64, case["N"]), r_max=case["R"], mixed=case["mixed"])
        st["eta"], st["rhs"] = ww.to_dev(eta), ww.to_dev(rhs)
    elif kind == "dtn_dd":
        eta, rhs = _dtn_host(case, seed)
        st["ctx"] = ww.Context(n_max=max(64, case["N"]), r_max=case["R"])
        st["eta"], st["rhs"] = ww.to_dev(eta), ww.to_dev(rhs)
        st["eta_lo"], st["rhs_lo"] = ww.to_dev(np.sin(1e3 * eta) * 1e-18), ww.to_dev(np.sin(7.0 * rhs) * 1e-17)
    elif kind in ("march", "f_only", "adjoint", "sdc"):
        st["ctx"], st["p"] = _shoot_context(case, seed)
    elif kind == "segments":
        st["ctx"] = ww.Context(n_max=case["N2"], r_max=case["M"] + 1)
        st["ctx"].shoot_setup(case["N"], INF, 0.0, 1.0, ww.to_dev(W.cosine_basis(case["N"], case["M"])),
                              ww.to_dev(np.zeros(2 * case["N"])))
        rng = np.random.default_rng([int(seed), 17])
        st["p"] = ww.to_dev(_modes(rng, case["a1"], case["M"]))
        # the shares of T/4 that the two segments' steps take, at the full march's step sizes
        t1, t2 = 0.2 * case["steps"] / case["full"], 0.8 * case["steps2"] / case["full2"]
        st["T"] = 2.0 * math.pi * (t1 + t2)
        st["segs"] = [dict(N=case["N"], nsteps=case["steps"], theta=t1 / (t1 + t2), rho=1.0),
                      dict(N=case["N2"], nsteps=case["steps2"], theta=1.0 - t1 / (t1 + t2), rho=case["rho"])]
    elif kind == "sdc_dd":
        rng = np.random.default_rng([int(seed), 17])
        N = case["N"]
        st["ctx"] = ww.Context(n_max=max(64, N), r_max=2)
        q = np.zeros(2 * N)
        p = _modes(rng, case["a1"], min(16, N // 3))
        q[:N] = W.cosine_basis(N, len(p))[:N] @ p
        st["q"] = ww.to_dev(q)
        st["q_lo"] = ww.to_dev(np.sin(1e3 * q) * 1e-18)
    elif kind == "batch":
        st["inst"] = _instances(case)
        made = [_shoot_context(c, int(seed) * 64 + i, stream=torch.cuda.Stream()) for i, c in enumerate(st["inst"])]
        st["ctxs"], st["ps"] = [m[0] for m in made], [m[1] for m in made]
        torch.cuda.synchronize()
    else:
        raise ValueError(kind)
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "dtn":
        st["ctx"].dtn_setup(st["eta"], _depth(case))
        out, mu = st["ctx"].dtn_solve_multi(st["rhs"], want_mu=True)
        return dict(out=out, mu=mu)
    if kind == "dtn_dd":
        st["ctx"].dtn_setup_dd(st["eta"], st["eta_lo"], _depth(case))
        oh, ol, mh, ml = st["ctx"].dtn_solve_multi_dd(st["rhs"], st["rhs_lo"], want_mu=True)
        return dict(out_hi=oh, out_lo=ol, mu_hi=mh, mu_lo=ml)
    if kind == "march":
        return st["ctx"].shoot_eval(st["p"], _period(case), case["steps"])
    if kind == "f_only":
        return st["ctx"].shoot_eval(st["p"], _period(case), case["steps"], jacobian=False)
    if kind == "adjoint":
        return st["ctx"].shoot_adjoint(st["p"], _period(case), case["steps"], case["ckpt"])
    if kind == "segments":
        return st["ctx"].shoot_eval_segments(st["p"], st["T"], st["segs"])
    if kind == "sdc":
        return st["ctx"].shoot_eval_sdc(st["p"], _period(case), case["steps"])
    if kind == "sdc_dd":
        return st["ctx"].shoot_eval_sdc_dd(case["N"], _depth(case), case["tau"], 1.0, st["q"], st["q_lo"],
                                           _period(case), case["steps"])
    if kind == "batch":
        return ww.shoot_eval_batch(st["ctxs"], st["ps"], [_period(c) for c in st["inst"]],
                                   [c["steps"] for c in st["inst"]])
    raise ValueError(kind)


# ----- the work a pass cannot do without ----------------------------------------------

def _stage_flops(N, R):
    """One stage: the factorisation of A, the solve and the product with Gm for R columns."""
    return 2.0 / 3.0 * N ** 3 + 4.0 * N * N * R


def work(case):
    kind = case["kind"]
    if kind == "dtn":
        N, R = case["N"], case["R"]
        return dict(bytes=8.0 * (N + 3 * N * R), flops=_stage_flops(N, R))
    if kind == "dtn_dd":
        # a double-double multiply-add counts 29 operations; residual and Gm products
        N, R = case["N"], case["R"]
        return dict(bytes=16.0 * (N + 3 * N * R), flops=2.0 / 3.0 * N ** 3 + 29.0 * 2.0 * N * N * R)
    if kind == "march":
        N, M = case["N"], case["M"]
        return dict(bytes=8.0 * (M + 2 * N * M + N * (M + 2)), flops=STAGES * case["steps"] * _stage_flops(N, M + 1))
    if kind == "f_only":
        N = case["N"]
        return dict(bytes=8.0 * (case["M"] + 4 * N), flops=STAGES * case["steps"] * _stage_flops(N, 1))
    if kind == "adjoint":
        N = case["N"]
        return dict(bytes=8.0 * (2 * case["M"] + 2 * N * case["M"]),
                    flops=STAGES * case["steps"] * (_stage_flops(N, 1) + 4.0 * N * N))
    if kind == "segments":
        M = case["M"]
        return dict(bytes=8.0 * (M + 2 * case["N"] * M + case["N2"] * (M + 2)),
                    flops=STAGES * (case["steps"] * _stage_flops(case["N"], M + 1) +
                                    case["steps2"] * _stage_flops(case["N2"], M + 1)))
    if kind == "sdc":
        N, M = case["N"], case["M"]
        return dict(bytes=8.0 * (M + 2 * N * M + N * (M + 2)),
                    flops=SDC_EVALS * case["steps"] * _stage_flops(N, M + 1))
    if kind == "sdc_dd":
        N = case["N"]
        return dict(bytes=16.0 * 6 * N, flops=SDC_EVALS * case["steps"] * (2.0 / 3.0 * N ** 3 + 29.0 * 2.0 * N * N))
    if kind == "batch":
        ws = [work(c) for c in _instances(case)]
        return dict(bytes=sum(w["bytes"] for w in ws), flops=sum(w["flops"] for w in ws))
    raise ValueError(kind)


# ----- the same results in plain 64-bit torch -----------------------------------------

class _Wave:
    """Boundary-integral DtN, right-hand sides and their variations in float64 torch."""

    def __init__(self, N, h, tau, dev):
        self.N, self.h, self.tau, self.dev = N, h, tau, dev
        a = torch.arange(N, dtype=torch.float64, device=dev) * (2.0 * math.pi / N)
        d = a[:, None] - a[None, :]
        self.sn, self.cs = torch.sin(d), torch.cos(d)
        self.sh2 = torch.sin(0.5 * d) ** 2
        self.c0 = torch.where(torch.eye(N, dtype=torch.bool, device=dev), torch.zeros_like(d),
                              0.5 / torch.tan(0.5 * d + torch.eye(N, dtype=torch.float64, device=dev)))
        k = torch.arange(N // 2 + 1, dtype=torch.float64, device=dev)
        self.k = k.clone()
        self.k[-1] = 0.0
        self.sig = torch.exp(-36.0 * (k / (N // 2)) ** 36)

    def _mul(self, x, sym):
        return torch.fft.irfft(torch.fft.rfft(x, dim=0) * (sym if x.dim() == 1 else sym[:, None]), n=self.N, dim=0)

    def dx(self, x):
        return self._mul(x, 1j * self.k)

    def filt(self, x):
        return self._mul(x, self.sig.to(torch.complex128))

    def proj(self, x):
        return x - x.mean(dim=0)

    def half_h(self, x):
        """H of a derivative, halved: the caller passes mu; the result is H(mu')/2."""
        return self._mul(x, (0.5 * self.k).to(torch.complex128))

    def matrices(self, eta):
        N = self.N
        ex, exx = self.dx(eta), self.dx(self.dx(eta))
        s = eta + (self.h if math.isfinite(self.h) else 0.0)
        eye = torch.eye(N, dtype=torch.bool, device=self.dev)

        def cot(y, off):
            # cot((x + i y)/2) = (sin x - i sinh y) / (cosh y - cos x)
            den = 2.0 * (torch.sinh(0.5 * y) ** 2 + self.sh2)
            if off:
                den = torch.where(eye, torch.ones_like(den), den)
            return self.sn / den, -torch.sinh(y) / den

        re, im = cot(s[:, None] - s[None, :], True)
        K = 0.5 * (im + ex[None, :] * re)
        G = 0.5 * (re - ex[:, None] * im) - self.c0
        den = 1.0 + ex * ex
        K = torch.where(eye, torch.diag(-0.5 * exx / den), K)
        G = torch.where(eye, torch.diag(0.5 * exx * ex / den), G)
        if math.isfinite(self.h):
            re, im = cot(s[:, None] + s[None, :], False)
            K = K - 0.5 * (im - ex[None, :] * re)
            G = G - 0.5 * (re - ex[:, None] * im)
        return 0.5 * torch.eye(N, dtype=torch.float64, device=self.dev) + K / N, G / N, ex

    def dtn(self, A, G, psi):
        mu = torch.linalg.solve(A, psi)
        return self.half_h(mu) + G @ self.dx(mu), mu

    def rhs(self, q, Q):
        """Slopes of the state (eta, phi) and of its variations (2N x M, or None)."""
        N = self.N
        eta, phi = q[:N], q[N:]
        A, Gm, ex = self.matrices(eta)
        B = phi[:, None]
        ps = self.dx(phi)
        if Q is not None:
            # the base solve first: phi_y enters the variations' Dirichlet data
            lu = torch.linalg.lu_factor(A)
            solve = lambda b: torch.linalg.lu_solve(*lu, b)
        else:
            solve = lambda b: torch.linalg.solve(A, b)
        mu = solve(B)
        Gp = (self.half_h(mu) + Gm @ self.dx(mu))[:, 0]
        den = 1.0 + ex * ex
        u, v = (ps - ex * Gp) / den, (ex * ps + Gp) / den
        pt = v * Gp - 0.5 * u * u - 0.5 * v * v - eta
        if self.tau:
            pt = pt + self.tau * self.dx(ex / torch.sqrt(den))
        k = torch.cat([self.filt(Gp), self.filt(self.proj(pt))])
        if Q is None:
            return k, None
        e, p = Q[:N], Q[N:]
        psi = p - v[:, None] * e
        mu = solve(psi)
        Gd = self.half_h(mu) + Gm @ self.dx(mu)
        et = Gd - self.dx(e * u[:, None])
        dv = -e * (u * v)[:, None]
        if self.tau:
            dv = dv + self.tau * self.dx(e) / (den * torch.sqrt(den))[:, None]
        pt = self.dx(dv) - u[:, None] * self.dx(psi) + v[:, None] * Gd - e
        return k, torch.cat([self.filt(et), self.filt(self.proj(pt))])


def _exact_march(case, seed, cols, grad=False):
    N, M, steps = case["N"], case["M"], case["steps"]
    # seconds: about 8 ms a stage at N = 256, growing with the dense solves
    if STAGES * steps * (4e-3 + 12e-3 * (N / 512.0) ** 2) > 15.0:
        return None
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    a, b, _ = ww.dop853()
    wv = _Wave(N, _depth(case), case["tau"], dev)
    basis = torch.as_tensor(W.cosine_basis(N, M), device=dev)
    q = basis @ torch.as_tensor(_march_host(case, seed), device=dev)
    Q = basis.clone() if cols else None
    T = _period(case)
    dt = T / (4.0 * steps)
    filt2 = lambda z: torch.cat([wv.filt(z[:N]), wv.filt(z[N:])])
    for _ in range(steps):
        ks, Ks = [], []
        for s in range(len(b)):
            y = q + sum((dt * a[s, j]) * ks[j] for j in range(s) if a[s, j] != 0.0)
            Y = Q + sum((dt * a[s, j]) * Ks[j] for j in range(s) if a[s, j] != 0.0) if cols else None
            k, K = wv.rhs(y, Y)
            ks.append(k)
            Ks.append(K)
        q = filt2(q + sum((dt * b[s]) * ks[s] for s in range(len(b))))
        if cols:
            Q = filt2(Q + sum((dt * b[s]) * Ks[s] for s in range(len(b))))
    w = 1.0 / math.sqrt(N)
    r = w * q[N:]
    d = 0.25 * w * wv.rhs(q, None)[0][N:]
    f = float(0.5 * (r @ r))
    if grad:
        return dict(grad=(w * Q[N:]).T @ r, dfdT=float(r @ d), f=f)
    return dict(r=r, J=w * Q[N:] if cols else None, drdT=d, f=f)


def exact(case, seed):
    kind = case["kind"]
    if kind == "dtn":
        eta, rhs = _dtn_host(case, seed)
        dev = "cuda" if torch.cuda.is_available() else "cpu"
        wv = _Wave(case["N"], _depth(case), 0.0, dev)
        A, G, _ = wv.matrices(torch.as_tensor(eta, device=dev))
        out, mu = wv.dtn(A, G, torch.as_tensor(rhs, device=dev))
        return dict(out=out, mu=mu)
    if kind in ("march", "f_only"):
        return _exact_march(case, seed, cols=kind == "march")
    if kind == "adjoint":
        return _exact_march(case, seed, cols=True, grad=True)
    if kind == "batch":
        outs = [_exact_march(c, int(seed) * 64 + i, cols=True) for i, c in enumerate(_instances(case))]
        return [dict(r=None, J=None, drdT=None, f=None) if o is None else o for o in outs]
    return None   # mapped meshes, SDC15 and double-double: no short 64-bit form
