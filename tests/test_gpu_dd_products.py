"""The double-double products and the solve around them at the sizes where their launches
change: one, two, three and four columns per workgroup (k_dd_gemm), ragged last tiles, the
one-column form, padded grids (N < 64), right-hand sides at an 8-byte offset."""
import math

import numpy as np
import pytest

from paper_1210_5672_amd import workloads as W

pytestmark = pytest.mark.gpu


def _ww():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5672_amd import ww
    return ww, torch


@pytest.mark.parametrize("N,R", [(16, 3), (32, 1), (64, 1), (64, 2), (256, 7), (512, 1), (512, 33), (1024, 2), (1024, 64), (1024, 129)])
def test_flat_symbol_over_the_launch_shapes(N, R):
    """G cos(k x) = k tanh(k h) cos(k x).  Tolerance: a sum of N terms rounds to N 2^-104 at
    worst, the derivative multiplies that by up to N/2: N^2 2^-105 of the symbol."""
    ww, torch = _ww()
    import mpmath
    mpmath.mp.dps = 40
    h = 1.0
    print(f"N={N} R={R}", flush=True)
    ks = [1 + c % 7 for c in range(R)]
    cs = [mpmath.cos(2 * mpmath.pi * j / N) for j in range(N)]
    hi1 = np.array([float(v) for v in cs])
    lo1 = np.array([float(v - mpmath.mpf(float(v))) for v in cs])
    idx = [(k * np.arange(N)) % N for k in ks]
    hi, lo = np.stack([hi1[i] for i in idx], 1), np.stack([lo1[i] for i in idx], 1)
    ctx = ww.Context(n_max=N, r_max=R)
    ctx.dtn_setup_dd(ww.to_dev(np.zeros(N)), None, h)
    oh, ol = ctx.dtn_solve_multi_dd(ww.to_dev(np.ascontiguousarray(hi)), ww.to_dev(np.ascontiguousarray(lo)))
    oh, ol = oh.cpu().numpy(), ol.cpu().numpy()
    for c in sorted({0, R // 2, R - 1}):
        k = ks[c]
        sym = k * mpmath.tanh(k * h)
        err = max(abs(mpmath.mpf(oh[j, c]) + mpmath.mpf(ol[j, c]) - sym * cs[(k * j) % N]) for j in range(N)) / sym
        print(f"column {c}: {float(err):.2e}", flush=True)
        assert err < N * N * 2.0 ** -105 + 10 * math.exp(-2 * (N - k) * h)
    ctx.close()


@pytest.mark.parametrize("N,R", [(16, 1), (32, 3), (64, 1), (64, 5), (128, 2)])
def test_offset_and_missing_low_parts(N, R):
    """Right-hand sides at an 8-byte offset, and without their low part, give the bits of the
    aligned ones with explicit zeros."""
    ww, torch = _ww()
    print(f"N={N} R={R}", flush=True)
    eta, rhs = W.random_surface(N, seed=N, amp=0.05), np.ascontiguousarray(W.random_rhs(N, R, seed=2))
    ctx = ww.Context(n_max=64 if N < 64 else N, r_max=R)
    ctx.dtn_setup_dd(ww.to_dev(eta), None, 0.8)
    a = ww.to_dev(rhs)
    want = ctx.dtn_solve_multi_dd(a, torch.zeros_like(a), want_mu=True)
    buf = torch.zeros(N * R + 1, dtype=torch.float64, device="cuda")
    off = buf[1:].as_strided(a.shape, a.stride())
    off.copy_(a)
    for got in (ctx.dtn_solve_multi_dd(off, torch.zeros_like(a), want_mu=True),
                ctx.dtn_solve_multi_dd(a, None, want_mu=True)):
        for x, y in zip(got, want):
            assert torch.equal(x, y)
    ctx.close()
