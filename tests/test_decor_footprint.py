"""Device memory of the correlation reduction (fmc_footprint, on the host): rows
that a workgroup ranks in LDS need no ranking buffers in memory."""
import pytest

import workloads

fmc = pytest.importorskip("paper_2007_03847_amd")


@pytest.mark.parametrize("N,words", [(2000, 3), (20000, 3), (20001, 7)])
def test_ranking_buffers_only_for_long_rows(N, words):
    sc = workloads.multimachine(n_gen=4, n_dist=3, N=N, K=40, T=0.1)
    extra = fmc.footprint(dict(sc, sampler="lhs_decor"), "f64") - fmc.footprint(sc, "f64")
    per = extra / (3 * 40 * N)
    # scores (8 bytes), the score ranks, the inverse ranks and one word spare per
    # entry; longer rows four words more; covariance and factor below 1.6 bytes
    # per entry and slice here
    assert 8 + 4 * words <= per < 8 + 4 * words + 12
