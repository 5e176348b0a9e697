"""Correlation reduction at the edges of its 16-row blocks and of the row lengths
that decide how a row is ranked, against the FP64 oracle.

The ranks are integers decided in FP64 on both sides and agree bit for bit, as do
the rearranged values."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(fmc):
    return fmc.Context(0)


# one, two and many blocks with and without remainder, the largest design; rows
# ranked with their values in LDS (to 10200), without (to 20000) and in memory
@pytest.mark.parametrize("M,N", [(15, 40), (16, 17), (17, 300), (33, 200), (64, 500), (420, 1000),
                                 (1024, 1100), (3, 10200), (3, 10201), (5, 20000), (5, 20001)])
def test_decorrelate_blocks(ctx, M, N):
    _, oz = oracle.lhs(900 + M, M, N, 0)
    z = ctx.torch.tensor(oz, dtype=ctx.torch.float64, device=ctx.device)
    st = ctx.lhs_decorrelate(z)
    ez, er = oracle.lhs_decorrelate(oz)
    assert np.array_equal(st.cpu().numpy(), er)
    assert np.array_equal(z.cpu().numpy(), ez)


def test_decorrelate_dependent_rows_and_ties(ctx, fmc):
    """A row that repeats another is refused with the design left as it was; equal
    values in a row are ranked by the lower sample index."""
    _, x = oracle.lhs(4, 20, 200, 0)
    x[18] = x[3]
    z = ctx.torch.tensor(x, dtype=ctx.torch.float64, device=ctx.device)
    with pytest.raises(fmc.FmcError):
        ctx.lhs_decorrelate(z)
    assert np.array_equal(z.cpu().numpy(), x)
    y = np.round(oracle.lhs(6, 20, 200, 0)[1], 1) + 0.0
    z = ctx.torch.tensor(y, dtype=ctx.torch.float64, device=ctx.device)
    st = ctx.lhs_decorrelate(z).cpu().numpy()
    assert np.array_equal(np.sort(st, axis=1), np.tile(np.arange(200), (20, 1)))
    assert np.array_equal(np.sort(z.cpu().numpy(), axis=1), np.sort(y, axis=1))
