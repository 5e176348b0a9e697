"""Network reduction at the edges of its two forms: the one-workgroup form
(n_bus (n_bus + n_gen) <= 4096) and the blocked one (32 buses a block, tiles of
32 x 64), against the FP64 oracle."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(fmc):
    return fmc.Context(0)


# (machines, buses): few buses; both sides of the 4096 limit; whole and ragged blocks
# of 32 buses; trailing matrices that end inside, at and past a tile
@pytest.mark.parametrize("n,nb", [(1, 2), (2, 2), (1, 63), (2, 63), (13, 51), (14, 51), (32, 64),
                                  (31, 64), (33, 64), (1, 64), (5, 65), (40, 95), (64, 96),
                                  (33, 97), (100, 128)])
def test_kron_forms_match_oracle(ctx, n, nb):
    net = workloads.network(n, seed=1000 + n, n_bus=nb, n_branch=max(nb - 1, int(1.2 * nb)))
    a, b = ctx.kron_reduce(net), oracle.kron(net)
    # the bound of the existing reduction tests: 1e-12 of the largest entry
    assert np.abs(a - b).max() <= 1e-12 * np.abs(b).max()


@pytest.mark.parametrize("n,nb", [(3, 12), (3, 100)])
def test_kron_singular_network_is_refused(ctx, fmc, n, nb):
    """A bus without branch, load or machine: its row of Y_BB is zero."""
    net = workloads.network(n, seed=5, n_bus=nb - 1)
    net = dict(net, n_bus=nb, load_g=np.append(net["load_g"], 0.0),
               load_b=np.append(net["load_b"], 0.0))
    with pytest.raises(fmc.FmcError) as e:
        ctx.kron_reduce(net)
    assert e.value.code == fmc.EINVAL
