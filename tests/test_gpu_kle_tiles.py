"""The KLE path contraction at the edges of its wave tiles and of the workgroups of
four of them (either tile shape), and the design at the edges of a workgroup's
samples and of the tabulated permutation, against the FP64 oracle: FP64 paths to 1e-13 of
the largest path value, FP32 storage to half a unit in its last place (6e-8), strata
bit for bit, values to 1e-15 (the other tests' bar)."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(fmc):
    return fmc.Context(0)


@pytest.mark.parametrize("prec,bar", [("f64", 1e-13), ("f32", 1e-7)])
@pytest.mark.parametrize("P,K,N,C", [(1, 5, 1, 1), (1, 8, 32, 32), (2, 9, 33, 31), (3, 12, 31, 33),
                                     (1, 7, 65, 97), (5, 4, 64, 129), (3, 21, 250, 419), (5, 9, 6601, 128),
                                     (6, 5, 5503, 110), (4, 6, 8192, 97)])
def test_kle_wave_tiles(ctx, P, K, N, C, prec, bar):
    t, S = ctx.torch, 300
    g = t.Generator(device=ctx.device)
    g.manual_seed(N + C)
    z = t.randn(P * K, N, dtype=t.float64, device=ctx.device, generator=g)
    phi = ctx.basis("paper", K, S, S * 0.005)
    for c0 in (0, 2 * S + 1 - C):
        w = ctx.kle_paths(z, phi, P, K, C, c0=c0, precision=prec).cpu().numpy().astype(np.float64)
        ref = oracle.kle_paths(z.cpu().numpy(), phi.cpu().numpy(), P, K, c0, C)
        assert np.abs(w - ref).max() <= bar * np.abs(ref).max()


@pytest.mark.parametrize("N", [1, 2, 3, 255, 2047, 2048, 2049, 65536, 65537, 262144, 262145])
@pytest.mark.parametrize("sampler", ["lhs", "srs"])
def test_design_sizes(ctx, N, sampler):
    st, z = ctx.lhs(seed=N, M=2, N=N, sampler=sampler)
    ost, oz = oracle.lhs(N, 2, N, 0 if sampler == "lhs" else 1)
    assert np.array_equal(st.cpu().numpy(), ost)
    assert np.all(np.abs(z.cpu().numpy() - oz) <= 1e-15 * np.maximum(1.0, np.abs(oz)))
