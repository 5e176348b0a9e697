"""Classical requests served beside a flux-decay request: their results are those
they have alone, bit for bit, and they advance by the steps of two of their halved
default chunks in a tick."""
import time

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(fmc):
    return fmc.Context(0)


def _np(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("prec", ["f32", "bf16x3"])
def test_mix_keeps_the_bits(ctx, prec):
    """Lane and team classes; horizons that end in the first and in the second chunk
    of a tick, one below the chunk, and a chunk of the caller's."""
    fd = workloads.fluxdecay(n_gen=20, n_dist=3, N=700, K=12, T=0.5)
    scs = [workloads.multimachine(n_gen=n, n_dist=3, N=N, K=12, T=S * 0.005, net_seed=n)
           for n, N, S in [(6, 300, 450), (12, 500, 430), (20, 333, 500), (45, 200, 60), (33, 400, 101)]]
    chunk = [0, 0, 0, 0, 37]
    alone = [ctx.submit(s, precision=prec, time_chunk=c).wait() for s, c in zip(scs, chunk)]
    fd_alone = ctx.submit(fd, precision=prec).wait()
    h = ctx.submit(fd, precision=prec)
    hs = [ctx.submit(s, precision=prec, time_chunk=c) for s, c in zip(scs, chunk)]
    mix = [x.wait() for x in hs]
    for a, b in zip(alone + [fd_alone], mix + [h.wait()]):
        assert np.array_equal(_np(a["mean"]), _np(b["mean"]))
        assert np.array_equal(_np(a["var"]), _np(b["var"]))


def test_two_chunks_in_a_tick_beside_flux_decay(ctx):
    """800 steps are eight chunks of 100: four ticks beside a flux-decay request of
    seven (12 steps each), so the classical request is done before it."""
    fd = workloads.fluxdecay(n_gen=100, n_dist=4, N=20000, K=20, T=84 * 0.005)
    sc = workloads.multimachine(n_gen=12, n_dist=3, N=300, K=12, T=4.0, net_seed=3)
    ctx.submit(sc).wait()  # the server runs
    t0 = time.perf_counter()
    h = ctx.submit(fd)
    t1 = time.perf_counter()
    c = ctx.submit(sc)
    done = t1 + c.wait()["report"]["latency_s"], t0 + h.wait()["report"]["latency_s"]
    assert done[0] < done[1]
