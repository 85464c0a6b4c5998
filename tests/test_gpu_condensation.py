"""The elimination of velocities and biases ahead of the reduced pose system,
at the sizes where its segments change: the shortest windows (a segment of one
and two keyframes, the middle keyframe without a neighbour on either side), the
longest segments, separators taken for the padding of the last tile or not,
windows of the one-workgroup and of the tile factorisation, with the biases
solved, held and shared, held poses inside a segment, and one context that
alternates between the option sets on one workspace.

One FP64 step against the oracle, which solves the full system in its natural
order.  Both are exact up to rounding, 1e-16 times the condition of the
Jacobi-scaled system (below 1e7 for these windows): 1e-8 relative per group, as
for every other FP64 step.
"""
import numpy as np
import pytest

from oracle import normal_eq as ne
from oracle import solve as osolve
from paper_2512_02293_amd import synth

pytestmark = pytest.mark.gpu
TOL = 1e-8
GROUPS = {"dtheta": slice(0, 3), "dp": slice(3, 6), "dv": slice(6, 9), "dbg": slice(9, 12), "dba": slice(12, 15)}


@pytest.fixture(scope="module")
def ctx():
    from paper_2512_02293_amd import binding
    c = binding.Context(0)
    yield c
    c.close()


def _problem(n, seed):
    return synth.make_problem(synth.SceneConfig(n_kf=n, H=9, W=11, k_out=min(4, n - 1), gap_range=(5, 25)), seed)


def _step(ctx, prob, mode, ws=None, **kw):
    import torch
    from paper_2512_02293_amd import binding
    o = binding.make_opts(bias_mode=mode, **kw)
    dp = binding.DeviceProblem(prob)
    imu = ctx.imu_preintegrate(dp.off, dp.gyro, dp.accel, dp.imu_dt, dp.bias_hat, dp.noise)
    nb = ctx.workspace_size(dp.cam, prob.n_kf, dp.ii, dp.jj, o)
    if ws is None:
        ws = torch.empty(nb, dtype=torch.uint8, device="cuda:0")
    assert ws.numel() == nb                    # every option set of a shape fits the same workspace
    dxi = torch.full((prob.n_kf, 15), 7.0, dtype=torch.float64, device="cuda:0")
    dd = torch.zeros_like(dp.invdepth)
    ctx.solve(dp.cam, dp.pose, dp.vel, dp.bias, dp.invdepth, dp.ii, dp.jj, dp.target, dp.weight, imu, o, 1, ws,
              dxi=dxi, dd=dd)
    cam, st, gr = osolve.from_problem(prob)
    oo = ne.Options(bias_fixed=mode == 1, bias_global=mode == 2, **kw)
    new, orep = osolve.step(cam, st, gr, oo)
    got = dxi.cpu().numpy()
    for g, sl in GROUPS.items():
        ref = orep["dxi"][:, sl]
        if np.linalg.norm(ref) == 0:
            assert not got[:, sl].any(), g
        else:
            assert np.linalg.norm(got[:, sl] - ref) <= TOL * np.linalg.norm(ref), g
    ref = orep["dd"]
    assert np.linalg.norm(dd.cpu().numpy() - ref) <= TOL * np.linalg.norm(ref)
    np.testing.assert_allclose(dp.vel.cpu().numpy(), new.v, rtol=0, atol=TOL * max(1.0, np.abs(new.v).max()))
    np.testing.assert_allclose(dp.bias.cpu().numpy(), new.b, rtol=0, atol=TOL)
    return ws


@pytest.mark.parametrize("n,mode,n_fixed", [(2, 0, 1), (2, 2, 1), (3, 0, 1), (3, 2, 1), (4, 1, 2), (5, 0, 3), (6, 0, 1),
                                            (7, 0, 1), (7, 2, 5), (10, 0, 1), (11, 2, 1), (13, 1, 1), (14, 0, 1),
                                            (25, 2, 2), (26, 0, 1), (52, 0, 15), (85, 0, 1), (90, 2, 1)])
def test_step_at_the_sizes_where_segments_change(ctx, n, mode, n_fixed):
    _step(ctx, _problem(n, 300 + n), mode, n_fixed=n_fixed)


def test_option_sets_of_one_shape_share_a_workspace(ctx):
    prob = _problem(39, 5)
    ws = _step(ctx, prob, 0)
    for kw in (dict(mode=2), dict(mode=0, use_imu=False), dict(mode=1), dict(mode=0, lm_lambda=1e-2)):
        _step(ctx, prob, ws=ws, **kw)
