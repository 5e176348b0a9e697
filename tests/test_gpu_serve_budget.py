"""The serving arena under a small memory budget: what is kept beside it (the
upload region of 16 MB) does not take from an arena that fits."""
import os

import pytest

import workloads

pytestmark = pytest.mark.gpu


def test_arena_of_64_mb_in_a_budget_of_84(fmc):
    old = os.environ.get("FMC_SERVE_ARENA_BYTES")
    os.environ["FMC_SERVE_ARENA_BYTES"] = str(64 << 20)
    try:
        ctx = fmc.Context(0, hbm_budget=84 << 20)
        sc = workloads.multimachine(n_gen=4, n_dist=2, N=200, K=10, T=0.2, net_seed=3)
        assert ctx.submit(sc).wait()["rc"] == 0
        ctx.close()
    finally:
        if old is None:
            os.environ.pop("FMC_SERVE_ARENA_BYTES")
        else:
            os.environ["FMC_SERVE_ARENA_BYTES"] = old
