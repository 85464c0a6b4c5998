"""Reduced systems beyond the one-workgroup Cholesky, whose keyframes are cut into
independent parts with rows skipped between them: chains of keyframes with and
without loop edges, just above the limit and well above it, with the shared
bias (which couples with every keyframe and stays out of the cut) and without
inertial factors.

One FP64 step against the oracle, which solves the full system in its natural
order: exact up to rounding times the condition of the scaled system, 1e-8
relative per group as for every other FP64 step.  The order of the sums is
fixed, so a repeated step is bitwise the same.
"""
import numpy as np
import pytest

from oracle import normal_eq as ne
from oracle import solve as osolve
from paper_2512_02293_amd import synth

pytestmark = pytest.mark.gpu
TOL = 1e-8


@pytest.mark.parametrize("n,loops,mode,imu", [(80, 0, 0, True), (87, 0, 0, False), (96, 24, 0, True), (96, 24, 2, True),
                                              (120, 40, 0, False), (150, 20, 1, True)])
def test_step_of_a_dissected_window(n, loops, mode, imu):
    import torch
    from paper_2512_02293_amd import binding
    prob = synth.make_problem(synth.SceneConfig(n_kf=n, H=6, W=8, k_out=4, n_loop=loops, gap_range=(5, 25)), 70 + n)
    ctx = binding.Context(0)
    try:
        out = []
        for _ in range(2):
            dp = binding.DeviceProblem(prob)
            o = binding.make_opts(bias_mode=mode, use_imu=imu)
            pre = ctx.imu_preintegrate(dp.off, dp.gyro, dp.accel, dp.imu_dt, dp.bias_hat, dp.noise)
            nb = ctx.workspace_size(dp.cam, prob.n_kf, dp.ii, dp.jj, o)
            ws = torch.empty(nb, dtype=torch.uint8, device="cuda:0")
            dxi = torch.zeros((prob.n_kf, 15), dtype=torch.float64, device="cuda:0")
            dd = torch.zeros_like(dp.invdepth)
            ctx.solve(dp.cam, dp.pose, dp.vel, dp.bias, dp.invdepth, dp.ii, dp.jj, dp.target, dp.weight, pre, o, 1, ws,
                      dxi=dxi, dd=dd)
            out.append((dxi.cpu().numpy(), dd.cpu().numpy()))
        assert all(np.array_equal(a, b) for a, b in zip(*out))
        cam, st, gr = osolve.from_problem(prob)
        _, rep = osolve.step(cam, st, gr, ne.Options(bias_fixed=mode == 1, bias_global=mode == 2, use_imu=imu))
        groups = [(out[0][0][:, s], rep["dxi"][:, s]) for s in (slice(0, 3), slice(3, 6), slice(6, 9), slice(9, 15))]
        for got, ref in groups + [(out[0][1], rep["dd"])]:
            assert np.linalg.norm(got - ref) <= TOL * np.linalg.norm(ref)
    finally:
        ctx.close()
