"""The vision assembly on either side of its rule (one edge per wave up to 8
edges per source, more slots above) and at the edges of its Gram tiles (6 k
rows: one, two and three tiles with and without padding), on maps smaller than
a chunk of 64 pixels, of one whole chunk, and ragged ones over several ranges.

One FP64 step against the oracle: exact up to rounding times the condition of
the scaled system, 1e-8 relative per group as for every other FP64 step.
"""
import numpy as np
import pytest

from oracle import normal_eq as ne
from oracle import solve as osolve
from paper_2512_02293_amd import synth

pytestmark = pytest.mark.gpu
TOL = 1e-8


@pytest.mark.parametrize("k,H,W", [(1, 9, 7), (2, 8, 8), (3, 5, 13), (5, 13, 17), (6, 16, 24), (7, 11, 13), (8, 8, 8),
                                   (8, 19, 23), (9, 8, 8), (9, 19, 23), (16, 7, 9)])
def test_step_at_out_degree(k, H, W):
    import torch
    from paper_2512_02293_amd import binding
    prob = synth.make_problem(synth.SceneConfig(n_kf=k + 2, H=H, W=W, k_out=k, gap_range=(5, 25)), 900 + k)
    deg = np.bincount(prob.ii, minlength=prob.n_kf)
    assert deg.max() == k
    ctx = binding.Context(0)
    try:
        dp = binding.DeviceProblem(prob)
        o = binding.make_opts(bias_mode=0)
        imu = ctx.imu_preintegrate(dp.off, dp.gyro, dp.accel, dp.imu_dt, dp.bias_hat, dp.noise)
        nb = ctx.workspace_size(dp.cam, prob.n_kf, dp.ii, dp.jj, o)
        ws = torch.empty(nb, dtype=torch.uint8, device="cuda:0")
        dxi = torch.zeros((prob.n_kf, 15), dtype=torch.float64, device="cuda:0")
        dd = torch.zeros_like(dp.invdepth)
        ctx.solve(dp.cam, dp.pose, dp.vel, dp.bias, dp.invdepth, dp.ii, dp.jj, dp.target, dp.weight, imu, o, 1, ws,
                  dxi=dxi, dd=dd)
        cam, st, gr = osolve.from_problem(prob)
        _, rep = osolve.step(cam, st, gr, ne.Options())
        for got, ref in ((dxi.cpu().numpy()[:, :6], rep["dxi"][:, :6]), (dxi.cpu().numpy()[:, 6:], rep["dxi"][:, 6:]),
                         (dd.cpu().numpy(), rep["dd"])):
            assert np.linalg.norm(got - ref) <= TOL * np.linalg.norm(ref)
    finally:
        ctx.close()
