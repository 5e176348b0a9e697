"""A path that is not finite stays with its sample: the others stay where they are,
to the bars of the other tests (FP64 1e-10, FP32 2e-3 of an output's largest value: an
angle that is not finite sends its neighbours to the general form of sin and cos), and
the report counts that sample alone.

The lanes (of a trajectory or a team) that own no process load some path value all
the same; whatever it is must not reach their trajectory."""
import ctypes as C

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(fmc):
    return fmc.Context(0)


def _np(t):
    return t.detach().cpu().numpy()


def designs(ctx, sc, bad):
    """The scenario's design, and the same with one value of process 0's in
    sample 0 replaced."""
    M = len(sc["dist"]["gen"]) * int(sc["K"])
    _, z = ctx.lhs(seed=5, M=M, N=int(sc["N"]))
    zb = z.clone()
    zb[1, 0] = bad
    return z, zb


def check(fmc, run, sc, bad, ctx, bar):
    z, zb = designs(ctx, sc, bad)
    a, b = run(z), run(zb)
    assert a["report"]["n_nonfinite"] == 0
    assert b["rc"] == fmc.ENONFINITE
    assert b["report"]["n_nonfinite"] == 1 and b["report"]["first_nonfinite"] == 0
    assert not np.isfinite(_np(b["traj"])[0, -1]).all()
    ta, tb = _np(a["traj"])[1:], _np(b["traj"])[1:]
    assert (np.abs(ta - tb).max(axis=(0, 1)) <= bar * np.abs(ta).max(axis=(0, 1))).all()


BAR = {"f64": 1e-10, "f32": 2e-3}


# the lanes forms (the lane of a machine owning its process, and processes spread
# over the lanes), one trajectory per lane, teams
@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("n,prec,vid", [(10, "f64", -1), (10, "f32", -1), (10, "f64", 16), (10, "f32", 22),
                                        (2, "f64", -1), (12, "f64", -1), (40, "f64", -1), (33, "f32", -1)])
def test_run(ctx, fmc, n, prec, vid, bad):
    P = min(3, n - 1)
    sc = workloads.multimachine(n_gen=n, n_dist=P, N=40, K=6, T=0.1, net_seed=60 + n)
    sel = np.array([0, 1, 17, 39])
    check(fmc, lambda z: ctx.run(sc, precision=prec, variant=vid, traj_idx=sel, zeta_in=z,
                                 allow_nonfinite=True), sc, bad, ctx, BAR[prec])


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_run_general_processes(ctx, fmc, prec):
    sc = workloads.config2_general(N=30, K=6, T=0.1)
    sel = np.array([0, 1, 29])
    check(fmc, lambda z: ctx.run(sc, precision=prec, traj_idx=sel, zeta_in=z, allow_nonfinite=True),
          sc, np.nan, ctx, BAR[prec])


@pytest.mark.parametrize("n,vid", [(9, -1), (12, 17), (40, 12), (20, 14)])
def test_batch(ctx, fmc, n, vid):
    prec = "bf16x3" if vid == 14 else "f32"
    sc = workloads.multimachine(n_gen=n, n_dist=3, N=70, K=6, T=0.1, net_seed=60 + n)

    def run(z):
        keep = fmc._Keep()
        sysd, dist, par, _ = fmc.scenario_structs(sc, prec, vid, 0, z, keep=keep)
        arr = (fmc.Scenario * 1)(fmc.Scenario(C.pointer(sysd), C.pointer(dist), C.pointer(par)))
        out, res = fmc._outputs_for(ctx, sc, np.array([0, 1, 65, 69]), keep)
        rc = fmc._lib.fmc_run_batch(ctx._h, 1, arr, (fmc.Outputs * 1)(out))
        assert rc in (0, fmc.ENONFINITE)
        return dict(rc=rc, traj=res["traj"], report=res["report"].as_dict())

    check(fmc, run, sc, np.nan, ctx, BAR["f32"])
