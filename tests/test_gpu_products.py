"""Products with the inverse for several columns (k_gemm_rm) at the edges of their tiles and of
the waves' split of the inner index: fewer chunks than waves, remainders of the chunk ring,
ragged and single columns per tile, both tile widths, both precision forms.

Tolerance: as for the inverse itself, N eps cond with cond <= 3 twice and G's largest
wavenumber relative to its own size: 1e-12 up to N = 2048."""
import numpy as np
import pytest

from oracle import ww_oracle as O
from paper_1210_5672_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = 1e-12


@pytest.mark.parametrize("mixed", [False, True])
@pytest.mark.parametrize("N", [16, 64, 128, 192, 324, 432, 576, 1024])
def test_column_products_at_tile_edges(N, mixed):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5672_amd import ww
    Rs = (2, 15, 16, 17, 31, 32, 33, 65)
    eta, rhs = W.random_surface(N, seed=N, amp=0.04), W.random_rhs(N, max(Rs), seed=N + 1)
    ref, mref = O.DtN(eta, 0.9).apply(rhs)
    ctx = ww.Context(n_max=max(N, 64), r_max=max(Rs), mixed=mixed)
    ctx.dtn_setup(ww.to_dev(eta), 0.9)
    for R in Rs:
        for rows in (16, 32):
            print(f"N={N} R={R} mixed={mixed} rows={rows}", flush=True)
            ctx.set_tuning(gemm_rows=rows)
            out, mu = ctx.dtn_solve_multi(ww.to_dev(np.asfortranarray(rhs[:, :R])), want_mu=True)
            eo = np.abs(out.cpu().numpy() - ref[:, :R]).max() / np.abs(ref).max()
            em = np.abs(mu.cpu().numpy() - mref[:, :R]).max() / np.abs(mref).max()
            assert max(eo, em) < TOL and ctx.fallbacks() == 0
    ctx.close()
