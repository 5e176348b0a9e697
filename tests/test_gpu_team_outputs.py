"""The team integrator against the lanes form, output by output: FP64 statistics and
trajectories within 1e-10 of each output's own largest value, machines that hardly move
(the network's H = 500 s equivalent) included.  Both integrate deviations from the
operating point, so the bar needs no allowance for absolute angles."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(fmc):
    return fmc.Context(0)


def _np(t):
    return t.detach().cpu().numpy()


# (machines, team, lanes form); full and ragged blocks of eight machines
@pytest.mark.parametrize("n,team,lanes", [(11, 34, 30), (16, 34, 30), (17, 35, 31), (24, 35, 31), (31, 36, 32),
                                          (33, 37, 33), (40, 37, 33), (47, 38, 33), (50, 39, 33)])
def test_every_output(ctx, n, team, lanes):
    sc = workloads.multimachine(n_gen=n, n_dist=min(8, n - 1), N=37, K=10, T=0.3, net_seed=600 + n)
    sel = np.array([0, 15, 16, 36])
    a = ctx.run(sc, variant=team, traj_idx=sel)
    b = ctx.run(sc, variant=lanes, traj_idx=sel)
    m, v = _np(b["mean"]), _np(b["var"])
    sd = np.sqrt(v.max(axis=0))
    scale = np.maximum(np.abs(m).max(axis=0), sd)
    assert (sd > 0).all()
    assert (np.abs(_np(a["mean"]) - m).max(axis=0) <= 1e-10 * scale).all()
    assert (np.abs(_np(a["var"]) - v).max(axis=0) <= 1e-10 * sd * sd).all()
    t = _np(b["traj"])
    assert (np.abs(_np(a["traj"]) - t).max(axis=(0, 1)) <= 1e-10 * np.abs(t).max(axis=(0, 1))).all()
