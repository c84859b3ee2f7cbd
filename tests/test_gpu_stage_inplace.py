"""The general transforms in place in the base chain of a lagged-factor march
(k_base_stage): the sizes that are neither 2^a nor 3 2^a and whose seven work buffers do not
fit in LDS, 1728 = 2^6 3^3 and 1944 = 2^3 3^5, with and without tension, on the uniform and on
a mapped grid, against the oracles.

One step: r, the base chain's output.  Tolerance: 1e-12 relative, the bar of the other
sizes: 12 stages of rounding at N = 1944 are of the order N eps = 5e-13."""
import math

import numpy as np
import pytest

from oracle import mesh_oracle as MO
from oracle import ww_oracle as O
from paper_1210_5672_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = 1e-12


def _ww():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5672_amd import ww
    return ww


def _rel(a, b):
    return float(np.abs(a.cpu().numpy() - b).max() / np.abs(b).max())


@pytest.mark.parametrize("N,tau", [(1728, 0.0), (1728, 0.001), (1944, 0.0), (1944, 0.001)])
def test_uniform_grid(N, tau):
    ww = _ww()
    print(f"N={N} tau={tau}", flush=True)
    h, M = 0.8, 1
    basis, qf, p = W.cosine_basis(N, M), np.zeros(2 * N), np.array([0.05])
    qf[:N] = 0.02 * np.cos(2 * W.grid(N)) + 0.003 * np.sin(3 * W.grid(N))
    T = W.linear_period(h, tau) / 600.0
    ctx = ww.Context(n_max=N, r_max=M + 1)
    ctx.shoot_setup(N, h, tau, 1.0, ww.to_dev(basis), ww.to_dev(qf))
    out = ctx.shoot_eval(ww.to_dev(p), T, 1)
    assert ctx.fallbacks() == 0
    assert _rel(out["r"], O.shoot_eval(N, h, tau, 1.0, basis, qf, p, T, 1, jacobian=False)["r"]) < TOL
    ctx.close()


@pytest.mark.parametrize("N,tau", [(1728, 0.001), (1944, 0.0)])
def test_mapped_grid(N, tau):
    ww = _ww()
    print(f"mapped N={N} tau={tau}", flush=True)
    h, M = math.inf, 1
    basis, qf, p = W.cosine_basis(N, M), np.zeros(2 * N), np.array([0.03])
    T = 2.0 * math.pi / 600.0
    segs = [dict(N=N, nsteps=1, theta=1.0, rho=0.7, refine_at=0)]
    ctx = ww.Context(n_max=N, r_max=M + 1)
    ctx.shoot_setup(N, h, tau, 1.0, ww.to_dev(basis), ww.to_dev(qf))
    out = ctx.shoot_eval_segments(ww.to_dev(p), T, segs)
    assert ctx.fallbacks() == 0
    assert _rel(out["r"], MO.shoot_eval_segments(N, h, tau, 1.0, basis, qf, p, T, segs)["r"]) < TOL
    ctx.close()
