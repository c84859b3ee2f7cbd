"""A finite surface whose matrix is not: heights beyond the range of exp, and heights within
it whose pairwise products are not (infinities and NaN off the diagonal only).  Every
pivot is then NaN from some block on, which no comparison with the guard shows; the call reports a
non-finite matrix instead of returning NaN.  One block, several, and a padded grid; a solve
of the mixed form, whose refinement test fails first, when it factors again in FP64; and the
double-double set-up."""
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
    return ww


@pytest.mark.parametrize("amp", [750.0, 400.0])
@pytest.mark.parametrize("N", [16, 64, 96, 192])
def test_matrix_out_of_range_is_reported(N, amp):
    ww = _ww()
    print(f"N={N} amp={amp}", flush=True)
    ctx = ww.Context(n_max=max(N, 64), r_max=1)
    with pytest.raises(ww.WWError) as e:
        ctx.dtn_setup(ww.to_dev(amp * np.cos(W.grid(N))), math.inf)
    assert e.value.name == "WW_ENONFINITE"
    # the context is as good as new
    ctx.dtn_setup(ww.to_dev(0.05 * np.cos(W.grid(N))), math.inf)
    assert ctx.fallbacks() == 0
    assert np.isfinite(ctx.dtn_solve_multi(ww.to_dev(np.cos(W.grid(N)))).cpu().numpy()).all()
    ctx.close()


@pytest.mark.parametrize("N", [64, 192])
def test_matrix_out_of_range_is_reported_by_the_mixed_form(N):
    ww = _ww()
    print(f"mixed N={N}", flush=True)
    ctx = ww.Context(n_max=N, r_max=1, mixed=True)
    with pytest.raises(ww.WWError) as e:
        ctx.dtn_setup(ww.to_dev(400.0 * np.cos(W.grid(N))), math.inf)
        ctx.dtn_solve_multi(ww.to_dev(np.cos(W.grid(N))))
    assert e.value.name == "WW_ENONFINITE"
    ctx.close()


def test_matrix_out_of_range_is_reported_in_double_double():
    ww = _ww()
    N = 128
    print("dd", flush=True)
    ctx = ww.Context(n_max=N, r_max=1)
    with pytest.raises(ww.WWError) as e:
        ctx.dtn_setup_dd(ww.to_dev(400.0 * np.cos(W.grid(N))), None, math.inf)
    assert e.value.name == "WW_ENONFINITE"
    ctx.close()


def test_small_pivots_still_take_the_pivoted_form(monkeypatch):
    """A guard above every pivot: the redo with row interchanges, not a non-finite report."""
    ww = _ww()
    N = 192
    print("guard", flush=True)
    eta, rhs = W.random_surface(N, seed=3, amp=0.05), W.random_rhs(N, 2, seed=4)
    a = ww.Context(n_max=N, r_max=2)
    a.dtn_setup(ww.to_dev(eta), 0.9)
    ref = a.dtn_solve_multi(ww.to_dev(rhs)).cpu().numpy()
    monkeypatch.setenv("WW_PIVOT_GUARD", "1.0")
    b = ww.Context(n_max=N, r_max=2)
    b.dtn_setup(ww.to_dev(eta), 0.9)
    assert b.fallbacks() == ww.WW_FB_PIVOTED | ww.WW_FB_FP64
    # two inverses of a matrix with cond(A) <= 3: N eps cond each, times G's largest mode
    assert np.abs(b.dtn_solve_multi(ww.to_dev(rhs)).cpu().numpy() - ref).max() < 1e-12 * np.abs(ref).max()
    a.close()
    b.close()
