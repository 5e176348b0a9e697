"""The design on both sides of the rule that decides between a tabulated and a
computed stratum permutation, against the FP64 oracle: strata bit for bit, values to
1e-15 (the other tests' bar); and the time of the sizes that the tables do not pay for."""
import time

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(fmc):
    return fmc.Context(0)


# M 4^h below and at the limits: 2^18 for N <= 1024, 3 * 2^18 above; N = 4^h
@pytest.mark.parametrize("M,N", [(255, 1000), (256, 1000), (256, 1024), (191, 1025), (192, 1025), (192, 4096),
                                 (11, 20000), (12, 20000), (2, 262144), (3, 262144), (3, 262145)])
def test_design_either_form(ctx, M, N):
    st, z = ctx.lhs(seed=M + N, M=M, N=N)
    ost, oz = oracle.lhs(M + N, M, N, 0)
    assert np.array_equal(st.cpu().numpy(), ost)
    assert np.all(np.abs(z.cpu().numpy() - oz) <= 1e-15 * np.maximum(1.0, np.abs(oz)))


def test_few_long_rows_take_no_tables(ctx):
    """20 rows of 8000 walk less than the tables cost (measured 18 us, 32 with
    tables): less time than 60 rows (33 us), which the tables take."""
    def best(M):
        t = []
        for _ in range(20):
            ctx.torch.cuda.synchronize()
            s = time.perf_counter()
            for _ in range(20):
                ctx.lhs(seed=1, M=M, N=8000, want_strata=False)
            ctx.torch.cuda.synchronize()
            t.append(time.perf_counter() - s)
        return min(t)

    assert best(20) < 0.9 * best(60)
