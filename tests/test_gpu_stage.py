"""The base chain of a lagged-factor march in spectral form (k_base_stage, k_base_dtn) at the
edges of its size classes -- unrolled and general transforms, work buffers with scratch and
in place, one and several entries per thread, ragged row blocks -- with and without tension,
on the uniform and on a mapped grid, against the oracles.

Two steps of a march whose lagged solves converge (no fallback): r, the base chain's output.
Tolerance: 1e-12 relative, the bar of the short marches elsewhere: 24 stages of rounding at
N = 2048 are of the order N eps = 5e-13."""
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
    return float(np.abs(np.asarray(a) - b).max() / np.abs(b).max())


@pytest.mark.parametrize("rows", [4, 8])
@pytest.mark.parametrize("N,tau", [(16, 0.0), (48, 0.01), (64, 0.01), (128, 0.0), (256, 0.0), (256, 0.01),
                                   (384, 0.005), (512, 0.0), (768, 0.002), (972, 0.005), (1024, 0.0), (1458, 0.002), (1536, 0.0), (2048, 0.0)])
def test_spectral_base_chain(N, tau, rows):
    ww = _ww()
    print(f"N={N} tau={tau} rows={rows}", flush=True)
    h, M, steps = 0.8, 1, 2 if N <= 1024 else 1
    basis, qf = W.cosine_basis(N, M), np.zeros(2 * N)
    qf[:N] = 0.02 * np.cos(2 * W.grid(N)) + 0.003 * np.sin(3 * W.grid(N))
    T = W.linear_period(h, tau) * steps / 600.0
    ctx = ww.Context(n_max=max(N, 64), r_max=M + 1)
    ctx.set_tuning(dtn_rows=rows)
    ctx.shoot_setup(N, h, tau, 1.0, ww.to_dev(basis), ww.to_dev(qf))
    out = ctx.shoot_eval(ww.to_dev(np.array([0.05])), T, steps)
    ref = O.shoot_eval(N, h, tau, 1.0, basis, qf, np.array([0.05]), T, steps)
    assert ctx.fallbacks() == 0
    assert _rel(out["r"].cpu().numpy(), ref["r"]) < TOL
    ctx.close()


@pytest.mark.parametrize("N,tau", [(64, 0.0), (72, 0.01), (256, 0.0), (512, 0.005), (768, 0.0), (1296, 0.0), (1536, 0.0)])
def test_spectral_base_chain_on_a_mapped_grid(N, tau):
    ww = _ww()
    print(f"mapped N={N} tau={tau}", flush=True)
    h, M, steps = math.inf, 1, 1
    basis, qf, p = W.cosine_basis(N, M), np.zeros(2 * N), np.array([0.03])
    T = 2.0 * math.pi * steps / 600.0
    segs = [dict(N=N, nsteps=steps, theta=1.0, rho=0.7, refine_at=0)]
    ctx = ww.Context(n_max=max(N, 64), r_max=M + 1)
    ctx.shoot_setup(N, h, tau, 1.0, ww.to_dev(basis), ww.to_dev(qf))
    out = ctx.shoot_eval_segments(ww.to_dev(p), T, segs)
    ref = MO.shoot_eval_segments(N, h, tau, 1.0, basis, qf, p, T, segs)
    assert ctx.fallbacks() == 0
    assert _rel(out["r"].cpu().numpy(), ref["r"]) < TOL
    # the column: the derivatives raise each stage's rounding by up to N/2, twelve stages
    assert _rel(out["J"].cpu().numpy(), ref["J"]) < 12 * N * np.finfo(float).eps
    ctx.close()
