"""The block Gauss-Jordan inverse (csrc/ww_inv.hpp) by strips of a set length (WW_GJ_STRIP):
the strip length follows from the number of blocks and matrices otherwise, and few-block
matrices would only ever see one tile a task.  One tile, strips with a remainder, all tiles
but one and a whole row, at two, three and six blocks (one padded), one matrix and groups of
up to four that share their launches, both precision forms.

A strip only groups tiles: every tile takes the same products in the same order, so the
results are the same bits at every length; at one of them they are held against the oracle.
Tolerance there: the forward error is at most about N eps cond(A), cond(A) <= 3 on these
surfaces, times G's largest wavenumber relative to its own size."""
import numpy as np
import pytest

from oracle import ww_oracle as O
from paper_1210_5672_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = 1e-12
SIZES = [(128, 2), (192, 3), (324, 6)]


def _ww():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5672_amd import ww
    return ww


def _strips(nb):
    return sorted({1, 2, 3, 4, nb - 1, nb} - {0})


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("N,nb", SIZES)
def test_one_matrix(N, nb, mixed, monkeypatch):
    ww = _ww()
    eta, rhs = W.random_surface(N, seed=N, amp=0.04), W.random_rhs(N, 3, seed=N + 1)
    ref, mref = O.DtN(eta, 0.9).apply(rhs)
    first = None
    for s in (s for s in _strips(nb) if s <= nb):
        print(f"N={N} mixed={mixed} strip={s}", flush=True)
        monkeypatch.setenv("WW_GJ_STRIP", str(s))
        ctx = ww.Context(n_max=N, r_max=3, mixed=mixed)
        ctx.dtn_setup(ww.to_dev(eta), 0.9)
        out, mu = (t.cpu().numpy() for t in ctx.dtn_solve_multi(ww.to_dev(rhs), want_mu=True))
        assert ctx.fallbacks() == 0
        ctx.close()
        if first is None:
            first = out, mu
            assert np.abs(out - ref).max() < TOL * np.abs(ref).max()
            assert np.abs(mu - mref).max() < TOL * np.abs(mref).max()
        assert np.array_equal(out, first[0]) and np.array_equal(mu, first[1])


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("group", [1, 2, 3, 4])
@pytest.mark.parametrize("N,nb", SIZES)
def test_groups(N, nb, group, mixed, monkeypatch):
    """A march's groups: J comes from every stage's own inverse, r from the lagged ones."""
    ww = _ww()
    h, M, steps = 0.8, 2, 2
    basis, qf = W.cosine_basis(N, M), np.zeros(2 * N)
    qf[:N] = 0.02 * np.cos(2 * W.grid(N)) + 0.003 * np.sin(3 * W.grid(N))
    T = W.linear_period(h, 0.0) * steps / 600.0
    first = None
    for s in (s for s in _strips(nb) if s <= nb):
        print(f"N={N} group={group} mixed={mixed} strip={s}", flush=True)
        monkeypatch.setenv("WW_GJ_STRIP", str(s))
        ctx = ww.Context(n_max=N, r_max=M + 1, mixed=mixed)
        ctx.set_tuning(lu_group=group)
        ctx.shoot_setup(N, h, 0.0, 1.0, ww.to_dev(basis), ww.to_dev(qf))
        o = ctx.shoot_eval(ww.to_dev(np.array([0.05, 0.01])), T, steps)
        assert ctx.fallbacks() == 0
        got = [o[k].cpu().numpy() for k in ("r", "J", "drdT")]
        ctx.close()
        if first is None:
            first = got
            ref = O.shoot_eval(N, h, 0.0, 1.0, basis, qf, np.array([0.05, 0.01]), T, steps)
            assert np.abs(got[0] - ref["r"]).max() < TOL * np.abs(ref["r"]).max()
        assert np.isfinite(got[1]).all()
        assert all(np.array_equal(a, b) for a, b in zip(first, got))
