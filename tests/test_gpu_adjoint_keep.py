"""The adjoint with the whole march's factors kept against segments recomputed from
checkpoints (WW_ADJOINT_KEEP=0): the same launches on the same data, the same bits.  Segment
lengths that divide the steps, that leave a remainder, and one longer than the march."""
import numpy as np
import pytest

from paper_1210_5672_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,ckpt", [(48, 1), (48, 5), (96, 8), (128, 40)])
def test_kept_and_recomputed_factors_agree(N, ckpt, monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5672_amd import ww
    print(f"N={N} ckpt={ckpt}", flush=True)
    M, nsteps, h, tau = 3, N // 4, 1.0, 0.01   # (fewer steps leave the stable range)
    p = ww.to_dev(np.array([0.03, 0.004, -0.002]))
    out = {}
    for keep in ("0", "64"):
        monkeypatch.setenv("WW_ADJOINT_KEEP", keep)
        ctx = ww.Context(n_max=128, r_max=M + 1)
        ctx.shoot_setup(N, h, tau, 1.0, ww.to_dev(W.cosine_basis(N, M)), ww.to_dev(np.zeros(2 * N)))
        for _ in range(2):   # the second call finds the workspace in place
            out[keep] = ctx.shoot_adjoint(p, W.linear_period(h, tau), nsteps, ckpt)
        out[keep]["grad"] = out[keep]["grad"].cpu().numpy()
        ctx.close()
    a, b = out["0"], out["64"]
    assert np.array_equal(a["grad"], b["grad"]) and a["f"] == b["f"] and a["dfdT"] == b["dfdT"]
