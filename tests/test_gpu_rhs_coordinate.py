"""The coordinate that a non-finite right-hand side is reported at: behind those
of the matrix (15 per keyframe, 7 in the pose graph), whatever of the unknowns
the reduced system keeps and in whatever order.

An infinite target leaves every matrix entry finite and spoils the right-hand
side at the keyframes of its source: the source itself and its targets.
"""
import re

import numpy as np
import pytest

from paper_2512_02293_amd import synth

pytestmark = pytest.mark.gpu


def _check(err, code, per, n, touched):
    assert err.code == code
    at = int(re.search(r"coordinate (-?\d+)", str(err)).group(1))
    assert per * n <= at < 2 * per * n, at
    assert (at - per * n) // per in touched


@pytest.mark.parametrize("n,k,imu", [(5, 3, False), (24, 5, True), (24, 12, True), (90, 4, True), (100, 4, False)])
def test_window(n, k, imu):
    import torch
    from paper_2512_02293_amd import binding
    prob = synth.make_problem(synth.SceneConfig(n_kf=n, H=9, W=11, k_out=k, gap_range=(5, 25)), 5)
    src = n // 3
    e = np.flatnonzero(prob.ii == src)
    y, x = np.argwhere(prob.weight[e[0], 0] > 0)[0]
    prob.target[e[0], 0, y, x] = np.inf
    ctx = binding.Context(0)
    try:
        dp = binding.DeviceProblem(prob)
        o = binding.make_opts(use_imu=imu)
        pre = ctx.imu_preintegrate(dp.off, dp.gyro, dp.accel, dp.imu_dt, dp.bias_hat, dp.noise)
        ws = torch.empty(ctx.workspace_size(dp.cam, n, dp.ii, dp.jj, o), dtype=torch.uint8, device="cuda:0")
        with pytest.raises(binding.ViError) as ei:
            ctx.solve(dp.cam, dp.pose, dp.vel, dp.bias, dp.invdepth, dp.ii, dp.jj, dp.target, dp.weight, pre, o, 1, ws)
        _check(ei.value, binding.VI_ENONFINITE, 15, n, {src, *prob.jj[e].tolist()})
    finally:
        ctx.close()


@pytest.mark.parametrize("n", [8, 120])
def test_pose_graph(n):
    import torch
    from paper_2512_02293_amd import binding
    loops = [(1, n - 2), (n // 2, 0), (n - 1, 2)]
    rel = [(i, i + s) for s in (1, 2) for i in range(n - s)]
    prob = synth.make_pgba_problem(synth.SceneConfig(n_kf=n, H=9, W=11, k_out=1), 5, loops, rel)
    e = int(np.flatnonzero(prob.ii == n // 2)[0])
    prob.target[e, 1] = np.inf
    ctx = binding.Context(0)
    try:
        o = binding.make_opts()
        pg = binding.DevicePGBA(prob)
        ws = torch.empty(ctx.pgba_workspace_size(pg, o), dtype=torch.uint8, device="cuda:0")
        with pytest.raises(binding.ViError) as ei:
            ctx.pgba_solve(pg, o, 1, ws)
        _check(ei.value, binding.VI_ENONFINITE, 7, n, {n // 2, 0})
    finally:
        ctx.close()
