"""The LU group that runs is the one that was chosen: the launch sequences of a profiled
march counted per step, for a context that was given no group (its rule: four stages where
the lag is at least eight, two otherwise), for every group by ww_set_tuning, by
ww_set_tuning_fields and by the environment, and for other choices made beside it."""
import ctypes

import numpy as np
import pytest

from paper_1210_5672_amd import workloads as W

pytestmark = pytest.mark.gpu
STAGES, STEPS = 12, 3


def _whole_struct(ww, ctx, **fields):
    """ww_get_tuning, change, ww_set_tuning: every field is chosen."""
    t = ww.Tuning()
    assert ctx.lib.ww_get_tuning(ctx.ptr, ctypes.byref(t)) == 0
    for n, v in fields.items():
        setattr(t, n, v)
    assert ctx.lib.ww_set_tuning(ctx.ptr, ctypes.byref(t)) == 0


CASES = [("none", {}, None, 4), ("none, lag 6", {"lag": 6}, None, 2), ("none, rows", {"dtn_rows": 4}, None, 4),
         ("named", {"lu_group": 1}, None, 1), ("named", {"lu_group": 2}, None, 2), ("named", {"lu_group": 3}, None, 3),
         ("named", {"lu_group": 4}, None, 4), ("struct", {"lu_group": 2}, None, 2), ("struct", {}, None, 2),
         ("environment", {}, "2", 2), ("environment", {}, "3", 3)]


@pytest.mark.parametrize("how,fields,env,group", CASES)
def test_group_that_runs(how, fields, env, group, monkeypatch):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1210_5672_amd import ww
    print(how, fields, env, flush=True)
    N, M, h = 64, 2, 1.0
    if env:
        monkeypatch.setenv("WW_LU_GROUP", env)
    ctx = ww.Context(n_max=N, r_max=M + 1)
    assert ctx.tuning()["lu_group"] == (int(env) if env else 2)
    if how == "struct":
        _whole_struct(ww, ctx, **fields)
    elif fields:
        ctx.set_tuning(**fields)
    if "lu_group" in fields:
        assert ctx.tuning()["lu_group"] == fields["lu_group"]
    ctx.shoot_setup(N, h, 0.0, 1.0, ww.to_dev(W.cosine_basis(N, M)), ww.to_dev(np.zeros(2 * N)))
    ctx.profile(True)
    ctx.shoot_eval(ww.to_dev(np.array([0.02, 0.001])), W.linear_period(h, 0.0) * STEPS / 100, STEPS)
    assert ctx.fallbacks() == 0
    assert ctx.profile_stats(0)[1] == STEPS * STAGES // group
    ctx.close()
