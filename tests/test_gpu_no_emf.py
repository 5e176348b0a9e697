"""A machine without EMF (E = 0) that runs away: it gives the network nothing,
whatever its angle has become, and the others follow the oracle.

With H = 0.05 s, D = 0 and Pm = 100 pu its angle passes 7e5 rad in two seconds,
where a polynomial in the angle has long left the range of FP32.

Bars of the other integrators: FP64 1e-10 of the largest value of its kind (angles,
speeds, processes: the oracle integrates absolute angles and rounds them), FP32 1e-4
of an output's own largest mean, deviation or variance."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(fmc):
    return fmc.Context(0)


def _np(t):
    return t.detach().cpu().numpy()


def runaway(n, N=33):
    sc = workloads.multimachine(n_gen=n, n_dist=min(3, n - 1), N=N, K=8, T=2.0, net_seed=80 + n)
    dead = next(i for i in range(n) if i not in sc["dist"]["gen"])
    E, H, D = sc["E"].copy(), sc["H"].copy(), sc["D"].copy()
    E[dead], H[dead], D[dead] = 0.0, 0.05, 0.0
    Et = E * np.exp(1j * sc["delta0"])
    Pm = (Et * np.conj(oracle.kron(sc["net"]) @ Et)).real
    Pm[dead] = 100.0
    return dict(sc, E=E, H=H, D=D, Pm=Pm), dead


def check(r, o, n, dead, prec):
    assert r["report"]["n_nonfinite"] == 0
    keep = np.array([v for v in range(o["mean"].shape[1]) if v not in (dead, n + dead)])
    assert np.abs(_np(r["mean"])[:, dead]).max() > 7e5
    m, v = o["mean"][:, keep], o["var"][:, keep]
    sd = np.sqrt(v.max(axis=0))
    scale = np.maximum(np.abs(m).max(axis=0), sd)
    if prec == "f64":
        for kind in (keep < n, (keep >= n) & (keep < 2 * n), keep >= 2 * n):
            sd[kind], scale[kind] = sd[kind].max(), scale[kind].max()
    bar = 1e-10 if prec == "f64" else 1e-4
    assert (np.abs(_np(r["mean"])[:, keep] - m).max(axis=0) <= bar * scale).all()
    assert (np.abs(_np(r["var"])[:, keep] - v).max(axis=0) <= bar * sd * sd).all()


# one trajectory per lane, lanes per trajectory, teams: the bars of the other tests
@pytest.mark.parametrize("n,prec,vid", [(2, "f32", -1), (10, "f32", -1), (10, "f32", 16), (12, "f32", 34),
                                        (33, "f32", -1), (2, "f64", -1), (10, "f64", -1), (12, "f64", -1)])
def test_run(ctx, n, prec, vid):
    sc, dead = runaway(n)
    check(ctx.run(sc, precision=prec, variant=vid), oracle.run(sc), n, dead, prec)


@pytest.mark.parametrize("n,vid", [(9, -1), (12, 17), (40, 12)])
def test_batched_and_served(ctx, n, vid):
    sc, dead = runaway(n)
    o = oracle.run(sc)
    check(ctx.run_batch([sc], variant=vid)[0], o, n, dead, "f32")
    check(ctx.submit(sc, variant=vid).wait(), o, n, dead, "f32")
