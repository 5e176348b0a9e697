"""The lanes-per-trajectory integrator where its branches part: the lane of a
machine owning the machine's process, against processes spread over the lanes
(several at one machine, or more processes than lanes), with padding machines,
idle lanes and ragged tiles.

Bars of the other integrators: FP64 within 1e-10 of each output's scale (a mean's:
the larger of it and the standard deviation), FP32 within 1e-4."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu

OWN = [0, 2, 4, 1]       # one process at a machine at most
SHARED = [2, 2, 0, 2]    # several at one


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


@pytest.mark.parametrize("prec,bar", [("f64", 1e-10), ("f32", 1e-4)])
@pytest.mark.parametrize("gen", [OWN, SHARED])
@pytest.mark.parametrize("n,N,vid", [(5, 31, -1), (10, 25, -1), (10, 7, 18), (10, 33, 22), (9, 49, 24),
                                     (10, 40, 13), (10, 65, 16)])
def test_process_ownership(ctx, n, N, vid, gen, prec, bar):
    """Processes, a trip of a driven machine, and time chunks that keep the bits."""
    sc = workloads.multimachine(n_gen=n, n_dist=4, N=N, K=10, T=0.3, net_seed=20 + n)
    sc["dist"] = dict(sc["dist"], gen=np.array(gen, dtype=np.int32), xi0=np.linspace(-0.02, 0.04, 4))
    for s in (sc, dict(sc, event=dict(t=0.1, tripped=2))):
        r = ctx.run(s, precision=prec, variant=vid)
        c = ctx.run(s, precision=prec, variant=vid, time_chunk=7)
        o = oracle.run(s)
        assert mean_err(_np(r["mean"]), o["mean"], o["var"]) <= bar
        assert rel_err(_np(r["var"]), o["var"]) <= bar
        assert np.array_equal(_np(r["mean"]), _np(c["mean"]))
        assert np.array_equal(_np(r["var"]), _np(c["var"]))


@pytest.mark.parametrize("prec,bar", [("f64", 1e-10), ("f32", 1e-4)])
@pytest.mark.parametrize("n,vid", [(1, -1), (2, -1)])
def test_few_machines(ctx, n, vid, prec, bar):
    """A trajectory per lane, coefficients in registers (one and two machines), and
    angles on both sides of the small-angle form of sin and 1 - cos."""
    sc = workloads.smib(N=70, K=8, T=0.5) if n == 1 else \
        workloads.multimachine(n_gen=2, n_dist=1, N=70, K=8, T=0.5, net_seed=3)
    for scale in (1.0, 12.0):
        s = dict(sc, dist=dict(sc["dist"], sigma=scale * np.asarray(sc["dist"]["sigma"])))
        r, o = ctx.run(s, precision=prec, variant=vid), oracle.run(s)
        assert mean_err(_np(r["mean"]), o["mean"], o["var"]) <= bar
        assert rel_err(_np(r["var"]), o["var"]) <= bar
