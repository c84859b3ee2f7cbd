"""Marches of two contexts at the same time, from two host threads: the same bits as alone,
and a march whose caller's stream is held up does not hold up the other one's.

The second needs more hardware queues than HIP's default of four (two marches have more
streams than that, and streams that share a queue wait for each other whatever the library
does), a choice that a process makes before it starts: it runs in a process of its own."""
import os
import subprocess
import sys

import numpy as np
import pytest

from paper_1210_5672_amd import workloads as W

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _contexts(N=256, M=16, steps=12):
    import torch
    from paper_1210_5672_amd import ww
    w = W.c2()
    basis, qf = ww.to_dev(W.cosine_basis(N, M)), ww.to_dev(w.q_fixed)
    out = []
    for i in range(2):
        ctx = ww.Context(n_max=N, r_max=M + 1, stream=torch.cuda.Stream())
        ctx.shoot_setup(N, w.h, w.tau, w.g, basis, qf)
        p = ww.to_dev((1.0 + 0.1 * i) * w.params[:M])
        out.append((ctx, p, w.T * steps / w.nsteps, steps))
    torch.cuda.synchronize()
    return out


def _march(x, jac=True):
    ctx, p, T, steps = x
    o = ctx.shoot_eval(p, T, steps, jacobian=jac)
    assert ctx.fallbacks() == 0
    return [o["r"].cpu().numpy(), o["drdT"].cpu().numpy()] + ([o["J"].cpu().numpy()] if jac else [])


def _held_up(jac):
    """A march while the other context's stream waits behind a kernel of the caller's (0.4 s):
    its time in seconds."""
    import threading
    import time
    import torch
    xs = _contexts()
    for x in xs + xs:
        _march(x, jac)
    t0 = time.perf_counter()
    torch.cuda._sleep(10 ** 8)
    torch.cuda.synchronize()
    count = int(0.4 * 1e8 / (time.perf_counter() - t0))
    with torch.cuda.stream(xs[0][0]._stream):
        torch.cuda._sleep(count)
    th = threading.Thread(target=_march, args=(xs[0], jac))
    th.start()
    time.sleep(0.05)   # the other march is enqueued
    t0 = time.perf_counter()
    xs[1][0].shoot_eval(xs[1][1], xs[1][2], xs[1][3], jacobian=jac)
    t = time.perf_counter() - t0
    th.join()
    return t


@pytest.mark.parametrize("jac", [True, False])
def test_marches_at_the_same_time_keep_their_bits(jac):
    import threading
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"jacobian={jac}", flush=True)
    xs = _contexts()
    alone = [_march(x, jac) for x in xs]
    got = [[], []]
    th = [threading.Thread(target=lambda i=i: got[i].extend(_march(xs[i], jac) for _ in range(3))) for i in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for a, runs in zip(alone, got):
        assert len(runs) == 3
        for g in runs:
            assert all(np.array_equal(x, y) for x, y in zip(a, g))


@pytest.mark.parametrize("jac", [1, 0])
def test_a_held_up_march_does_not_hold_up_another(jac):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"jacobian={jac}", flush=True)
    code = f"import test_gpu_two_marches as t; print('SECONDS', t._held_up(bool({jac})))"
    env = dict(os.environ, GPU_MAX_HW_QUEUES="16")
    env["PYTHONPATH"] = os.pathsep.join([ROOT, os.path.join(ROOT, "tests"), env.get("PYTHONPATH", "")])
    run = subprocess.run([sys.executable, "-c", code], env=env, capture_output=True, text=True, timeout=90)
    assert run.returncode == 0, run.stderr[-2000:]
    t = float(run.stdout.split("SECONDS")[1])
    print(f"march beside a held-up one: {1e3 * t:.0f} ms", flush=True)
    assert t < 0.2   # it takes a few ms; held up, it would take the 0.35 s that are left of the wait


if __name__ == "__main__":
    print(_held_up(True), _held_up(False))
