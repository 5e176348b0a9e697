"""The team integrator (a tile of 16 trajectories per workgroup, eight machines
per wave, the network product on the matrix cores) against the FP64 oracle, at
the edges of its blocks of eight machines and tiles of 16 samples.

Bars of the other integrators: FP64 within 1e-10, FP32 mean/var within 1e-4.  The
scale of an FP64 statistic is the largest of its kind (angles, speeds, processes):
the oracle integrates absolute angles, so its own rounding is that of an angle of
order one, which for the statistics of a machine that hardly moves (the network's
H = 500 s equivalent) exceeds 1e-10 of their own size.  (FP64 variants of either
kind agree on those to 1e-14 and differ from the oracle by the same amount.)"""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

TEAM0 = 34  # first team variant: 16, 24, 32, 40, 48, 50 machines


@pytest.fixture(scope="module")
def ctx(fmc):
    return fmc.Context(0)


def _np(t):
    return t.detach().cpu().numpy()


def rel_err(a, b):
    num = np.abs(a - b).reshape(-1, a.shape[-1]).max(axis=0)
    den = np.abs(b).reshape(-1, b.shape[-1]).max(axis=0)
    return float((num / np.where(den == 0, 1, den)).max())


def mean_err(a, m, v):
    num = np.abs(a - m).max(axis=0)
    den = np.maximum(np.abs(m).max(axis=0), np.sqrt(np.abs(v)).max(axis=0))
    return float((num / np.where(den == 0, 1, den)).max())


def check(ctx, sc, prec, **kw):
    sel = np.array([0, int(sc["N"]) - 1])
    r = ctx.run(sc, precision=prec, traj_idx=sel, **kw)
    o = oracle.run(sc, want_traj=True)
    if prec == "f64":
        n = sc["n_gen"]
        for k in (slice(0, n), slice(n, 2 * n), slice(2 * n, None)):
            sd = np.sqrt(o["var"][:, k].max())
            scale = max(np.abs(o["mean"][:, k]).max(), sd)
            assert np.abs(_np(r["mean"])[:, k] - o["mean"][:, k]).max() <= 1e-10 * scale
            assert np.abs(_np(r["var"])[:, k] - o["var"][:, k]).max() <= 1e-10 * sd * sd
            t, ot = _np(r["traj"])[:, :, k], o["traj"][sel][:, :, k]
            assert np.abs(t - ot).max() <= 1e-10 * np.abs(ot).max()
    else:
        assert mean_err(_np(r["mean"]), o["mean"], o["var"]) <= 1e-4
        assert rel_err(_np(r["var"]), o["var"]) <= 1e-4
    return r


SIZES = [(11, 1, 16), (16, 8, 17), (17, 4, 15), (24, 5, 33), (25, 8, 2), (32, 3, 31), (33, 2, 48),
         (40, 8, 16), (41, 1, 40), (48, 7, 18), (49, 8, 17), (50, 8, 35)]


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("n,P,N", SIZES)
def test_team_sizes(ctx, n, P, N, prec):
    sc = workloads.multimachine(n_gen=n, n_dist=P, N=N, K=12, T=0.2, net_seed=300 + n)
    r = check(ctx, sc, prec, variant=TEAM0 + (n + 7) // 8 - 2)
    assert r["report"]["tile"] == 16


@pytest.mark.parametrize("n,N,prec,team", [(10, 40, "f64", False), (11, 40, "f64", True),
                                           (16, 12000, "f32", False), (16, 12001, "f32", True),
                                           (24, 1500, "f32", False), (24, 1501, "f32", True),
                                           (25, 20, "f32", True)])
def test_team_is_the_default_above_ten_machines(ctx, n, N, prec, team):
    sc = workloads.multimachine(n_gen=n, n_dist=2, N=N, K=8, T=0.05, net_seed=5)
    r = ctx.run(sc, precision=prec)
    assert (r["report"]["variant_id"] >= TEAM0) == team


# The batched and served forms: teams of two to eight waves, the ones of five and
# six in pairs (tiles of 32); full, ragged and single tiles, several tiles per item
BATCH = [(12, 3, 33), (16, 8, 16), (17, 2, 47), (24, 8, 31), (32, 4, 65), (33, 8, 32), (40, 1, 33),
         (41, 5, 31), (48, 8, 80), (49, 2, 17), (56, 8, 33), (57, 1, 15), (64, 8, 100)]


@pytest.mark.parametrize("n,P,N", BATCH)
def test_team_batched_and_served(ctx, n, P, N):
    vid = 17 if n <= 16 else 11 if n <= 32 else 12 if n <= 48 else 13
    sc = workloads.multimachine(n_gen=n, n_dist=P, N=N, K=9, T=0.25, net_seed=400 + n)
    o = oracle.run(sc)
    outs = [ctx.run_batch([sc], variant=vid)[0], ctx.submit(sc, variant=vid).wait(),
            ctx.submit(sc, variant=vid, time_chunk=17).wait(),
            ctx.run_batch([sc], variant=vid, time_chunk=17)[0]]
    for r in outs:
        assert r["report"]["variant_id"] == vid
        assert mean_err(_np(r["mean"]), o["mean"], o["var"]) <= 1e-4
        assert rel_err(_np(r["var"]), o["var"]) <= 1e-4
    # time chunks keep the bits
    assert np.array_equal(_np(outs[0]["mean"]), _np(outs[3]["mean"]))
    assert np.array_equal(_np(outs[0]["var"]), _np(outs[3]["var"]))


@pytest.mark.parametrize("vid,n", [(TEAM0, 1), (TEAM0, 3), (TEAM0 + 1, 10), (TEAM0 + 5, 50)])
def test_team_variant_by_id(ctx, vid, n):
    """A team variant asked for by id, with most of its machines padding."""
    sc = workloads.smib(N=37, K=8, T=0.3) if n == 1 else \
        workloads.multimachine(n_gen=n, n_dist=min(2, n - 1), N=37, K=8, T=0.2, net_seed=7)
    check(ctx, sc, "f64", variant=vid)


def test_team_several_processes_per_machine(ctx):
    sc = workloads.multimachine(n_gen=12, n_dist=8, N=40, K=10, T=0.2, net_seed=3)
    sc["dist"] = dict(sc["dist"], gen=np.array([5, 5, 5, 2, 2, 11, 0, 5], dtype=np.int32),
                      xi0=np.linspace(-0.05, 0.1, 8))
    check(ctx, sc, "f64")


def test_team_chunks_event_and_rrf(ctx):
    """Time chunks keep the bits; a generator trip and the RRF match the oracle."""
    sc = workloads.multimachine(n_gen=19, n_dist=4, N=50, K=10, T=0.4, net_seed=11)
    w = workloads.coi_frequency_weights(sc)
    trip = dict(sc, event=dict(t=0.1, tripped=int(sc["dist"]["gen"][1])))
    for s in (sc, trip):
        a = check(ctx, s, "f64", rrf_weights=w)
        b = ctx.run(s, precision="f64", rrf_weights=w, time_chunk=7)
        for k in ("mean", "var", "rrf"):
            assert np.array_equal(_np(a[k]), _np(b[k])), k
        o = oracle.run(s, want_traj=True)
        ref = oracle.rrf_rms(o["traj"], w, s["dt"])
        assert np.abs(_np(a["rrf"]) - ref).max() <= 1e-10 * np.abs(ref).max()


def test_team_counts_nonfinite_paths(ctx, fmc):
    sc = workloads.multimachine(n_gen=12, n_dist=2, N=20, K=8, T=0.5, net_seed=3)
    sc["dist"] = dict(sc["dist"], sigma=np.full(2, 1e200))
    r = ctx.run(sc, allow_nonfinite=True)
    assert r["rc"] == fmc.ENONFINITE and r["report"]["n_nonfinite"] == 20
    assert r["report"]["first_nonfinite"] == 0


def test_team_refuses_general_processes(ctx, fmc):
    sc = workloads.config2_general(N=20, T=0.1)
    with pytest.raises(fmc.FmcError) as e:
        ctx.run(sc, variant=TEAM0)
    assert e.value.code == fmc.EINVAL
    with pytest.raises(fmc.FmcError) as e:  # beyond 50 machines as before
        ctx.run(workloads.multimachine(n_gen=51, N=16, K=4, T=0.05))
    assert e.value.code == fmc.EINVAL
