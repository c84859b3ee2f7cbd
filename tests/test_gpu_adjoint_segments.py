"""The adjoint with the whole march's factors kept against segments recomputed from
checkpoints (WW_ADJOINT_KEEP=0), on grids of one and of several blocks, with and without the
pivoted fallback: the workspace that each takes shows that both forms ran, both give the
same bits, and those are the oracle's gradient.

Tolerance against the oracle: the bar of the other adjoint tests, 1e-12."""
import numpy as np
import pytest

from oracle import ww_oracle as O
from paper_1210_5672_amd import workloads as W

pytestmark = pytest.mark.gpu
TOL = 1e-12
MIB = 1 << 20


@pytest.mark.parametrize("N,ckpt,pivoted", [(48, 5, False), (96, 8, False), (128, 8, False), (128, 9, False),
                                            (192, 16, False), (96, 8, True)])
def test_kept_and_recomputed_factors_agree(N, ckpt, pivoted, monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5672_amd import ww
    print(f"N={N} ckpt={ckpt} pivoted={pivoted}", flush=True)
    M, nsteps, h, tau = 3, N // 4, 1.0, 0.01   # (fewer steps leave the stable range)
    basis, qf, p = W.cosine_basis(N, M), np.zeros(2 * N), np.array([0.03, 0.004, -0.002])
    T = W.linear_period(h, tau)
    if pivoted:
        monkeypatch.setenv("WW_PIVOT_GUARD", "1.0")   # above every pivot (about 0.5)
    Np = (N + 63) // 64 * 64
    slots = lambda steps: 8 * steps * 12 * (2 * Np * Np + 3 * N)   # bytes of the factors of so many steps
    out = {}
    for keep in ("0", "1024"):
        monkeypatch.setenv("WW_ADJOINT_KEEP", keep)
        ctx = ww.Context(n_max=max(N, 64), r_max=M + 1)
        ctx.shoot_setup(N, h, tau, 1.0, ww.to_dev(basis), ww.to_dev(qf))
        dp = ww.to_dev(p)
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        for call in range(2):   # the second call finds the workspace in place
            o = ctx.shoot_adjoint(dp, T, nsteps, ckpt)
            o["grad"] = o["grad"].cpu().numpy()
            if call == 0:
                taken = free - torch.cuda.mem_get_info()[0]
        assert ctx.fallbacks() == (ww.WW_FB_PIVOTED | ww.WW_FB_FP64 if pivoted else 0)
        # (beside the factors: checkpoints, work vectors, the pivoted form's matrix, torch's 2 MiB blocks)
        want = slots(nsteps if keep != "0" else ckpt)
        assert want <= taken + 2 * MIB and taken <= want + 16 * MIB, (taken / MIB, want / MIB)
        assert slots(nsteps) - slots(ckpt) > 18 * MIB or N == 48   # the two forms tell apart
        out[keep] = o
        ctx.close()
    a, b = out["0"], out["1024"]
    assert np.array_equal(a["grad"], b["grad"]) and a["f"] == b["f"] and a["dfdT"] == b["dfdT"]
    if N <= 128:
        ref, _ = O.shoot_gradient(O.shoot_eval(N, h, tau, 1.0, basis, qf, p, T, nsteps))
        assert np.linalg.norm(b["grad"] - ref) < TOL * np.linalg.norm(ref)
