"""Network reduction: which networks are refused as singular, and admittances far
from one, in the one-workgroup form (20 buses) and the blocked one (70 and 150)."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(fmc):
    return fmc.Context(0)


@pytest.mark.parametrize("nb,pair", [(20, (3, 4)), (20, (0, 19)), (70, (3, 4)), (70, (0, 69)), (150, (40, 41)),
                                     (150, (31, 32)), (150, (0, 149))])
def test_island_of_two_buses_is_refused(ctx, fmc, nb, pair):
    """Two buses that only a reactance joins: the pivot of the second cancels to
    zero exactly, in the same block of buses as the first or in a later one."""
    rest = np.array([b for b in range(nb) if b not in pair])
    for seed in range(24):
        net = workloads.network(4, seed=seed, n_bus=nb - 2)
        lg, lb = np.zeros(nb), np.zeros(nb)
        lg[rest], lb[rest] = net["load_g"], net["load_b"]
        island = dict(net, n_bus=nb, br_from=np.append(rest[net["br_from"]], pair[0]),
                      br_to=np.append(rest[net["br_to"]], pair[1]), br_r=np.append(net["br_r"], 0.0),
                      br_x=np.append(net["br_x"], 0.01 + 0.0037 * seed), br_b=np.append(net["br_b"], 0.0),
                      load_g=lg, load_b=lb, gen_bus=rest[net["gen_bus"]])
        with pytest.raises(fmc.FmcError) as e:
            ctx.kron_reduce(island)
        assert e.value.code == fmc.EINVAL


@pytest.mark.parametrize("nb", [20, 70, 150])
@pytest.mark.parametrize("e", [-520, -200, 200, 480])
def test_admittances_of_any_size(ctx, nb, e):
    """The reduction is linear in a common factor of all admittances: a power of two
    changes no digit that is not rounded away (bar of the other reduction tests)."""
    s = 2.0 ** e
    net = workloads.network(4, seed=nb, n_bus=nb)
    b = ctx.kron_reduce(net)
    a = ctx.kron_reduce(dict(net, br_r=net["br_r"] / s, br_x=net["br_x"] / s, load_g=net["load_g"] * s,
                             load_b=net["load_b"] * s, gen_xdp=net["gen_xdp"] / s))
    assert np.abs(a / s - b).max() <= 1e-12 * np.abs(b).max()
