"""The block Gauss-Jordan inverse (csrc/ww_inv.hpp) through dtn_setup / dtn_solve_multi at
the edges of its tiles and tasks: one block, two blocks, ragged and odd block counts, every
strip length from one tile to a whole row, both precision forms.

Tolerance: the solve's forward error is at most about N eps cond(A), cond(A) <= 3 on these
surfaces, and G multiplies it by at most the largest wavenumber relative to its own size:
1e-12 covers N = 2048 with a factor of two to spare."""
import numpy as np
import pytest

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


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("N,strips", [(16, (4,)), (64, (1, 4)), (72, (1, 2)), (128, (1, 16)), (192, (1, 2, 3)),
                                      (324, (1, 5, 16)), (1152, (2, 4)), (2048, (1, 4, 16))])
def test_inverse_at_tile_edges(N, strips, mixed):
    ww = _ww()
    eta, rhs = W.random_surface(N, seed=N, amp=0.04), W.random_rhs(N, 3, seed=N + 1)
    ref, mref = O.DtN(eta, 0.9).apply(rhs)
    ctx = ww.Context(n_max=max(N, 64), r_max=3, mixed=mixed)
    for s in strips:
        print(f"N={N} mixed={mixed} strip={s}", flush=True)
        ctx.set_tuning(blu_strip=s)
        ctx.dtn_setup(ww.to_dev(eta), 0.9)
        out, mu = ctx.dtn_solve_multi(ww.to_dev(rhs), want_mu=True)
        eo = np.abs(out.cpu().numpy() - ref).max() / np.abs(ref).max()
        em = np.abs(mu.cpu().numpy() - mref).max() / np.abs(mref).max()
        assert max(eo, em) < TOL and ctx.fallbacks() == 0
    ctx.close()


def test_nan_entry_does_not_pass_the_guard():
    """A non-finite surface is reported, not inverted."""
    ww = _ww()
    eta = W.random_surface(128, seed=1)
    eta[70] = np.nan
    ctx = ww.Context(n_max=128, r_max=1)
    with pytest.raises(ww.WWError) as e:
        ctx.dtn_setup(ww.to_dev(eta), float("inf"))
    assert e.value.name == "WW_ENONFINITE"
    ctx.close()
