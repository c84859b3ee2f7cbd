"""dtn_solve_multi_dd with outputs on top of its right-hand sides: in place, planes exchanged,
shifted by a few entries, and the density on top of the right-hand side: the bits of outputs
of their own.  Grids that are used as they are and one that is padded, one column (its own
product) and several."""
import ctypes

import numpy as np
import pytest

from paper_1210_5672_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,R", [(32, 3), (64, 1), (64, 5), (256, 4)])
def test_outputs_on_top_of_the_right_hand_sides(N, R):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5672_amd import ww
    print(f"N={N} R={R}", flush=True)
    ctx = ww.Context(n_max=max(N, 64), r_max=R)
    ctx.dtn_setup_dd(ww.to_dev(W.random_surface(N, seed=N, amp=0.05)), None, 0.8)
    n, pad = N * R, 6
    rhs = torch.as_tensor(np.ascontiguousarray(W.random_rhs(N, R, seed=2).T)).reshape(-1).to("cuda")
    low = rhs * 2.0 ** -60

    def solve(out_hi, out_lo, mu_hi=None, mu_lo=None):
        """Offsets into one buffer: rhs_hi at 0, rhs_lo at n + pad, room behind."""
        buf = torch.zeros(6 * (n + pad), dtype=torch.float64, device="cuda")
        buf[:n] = rhs
        buf[n + pad:2 * n + pad] = low
        at = lambda o: None if o is None else ctypes.c_void_p(buf.data_ptr() + 8 * o)
        torch.cuda.synchronize()
        rc = ctx.lib.dtn_solve_multi_dd(ctx.ptr, at(0), at(n + pad), R, at(out_hi), at(out_lo), at(mu_hi), at(mu_lo))
        torch.cuda.synchronize()
        assert rc == 0, ctx.lib.ww_last_error()
        return [buf[o:o + n].clone() for o in (out_hi, out_lo, mu_hi, mu_lo) if o is not None]

    a, b, c, d, e, f = (k * (n + pad) for k in range(6))
    want = solve(c, d, e, f)
    for where in ((a, b), (b, a), (a + 4, b), (a, b + pad // 2), (c, a, b, d), (c, d, a, b)):
        got = solve(*where)
        assert all(torch.equal(x, y) for x, y in zip(want, got)), where
    ctx.close()
