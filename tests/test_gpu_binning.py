"""Binning of loaded particles and their backward half step against the oracle's
loader: several chunks per load, the path of boxes with very many tiles, and a
second load into tiles that already hold particles."""
import numpy as np
import pytest

from tests import gpu_cases as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("dims,tile", [((16, 16, 16), (4, 4, 4)), ((13, 7, 5), (4, 4, 4)), ((9, 8, 11), (8, 4, 2)),
                                       ((32, 32, 20), (1, 1, 1))],
                         ids=["chunks", "ragged", "tile842", "many_tiles"])
def test_loads_are_binned_and_integrated_back(dims, tile, fp64):
    # b is random, so that the half step turns every momentum; loader and half
    # step tolerances as in the loader's own test
    rng = np.random.default_rng(5)
    cells = int(np.prod(dims))
    n_x, dt = 10.0, 0.5
    ppc = [round(9500 / cells, 3), round(700 / cells, 3)]
    npairs = [int(p * cells + 0.5) for p in ppc]
    _, b = G.random_fields(rng, cells, 0.0, 0.4)
    b = G.field_storage(b, fp64)
    s = G.sim(dims, n_x, 16.0, [sum(npairs)] * 2, fp64=fp64, tile=tile)
    s.set_fields(0, np.zeros(3 * cells), b)
    A, Bp = {"theta": 0.2, "gb": 0.3, "axis": 2}, {"theta": 0.7, "gb": 0.0, "axis": 0}
    for k in range(2):
        s.load(0, 0, 1, (0.2, 0.3, 2), (0.7, 0.0, 0), ppc[k], seed=9, stream=k)
        s.step(0)
    parts = G.oracle_loaded(dims, dt, n_x, 16.0, G.PAIR,
                            [dict(seed=9, stream=k, npairs=npairs[k], A=A, B=Bp) for k in range(2)], b=b)
    for sp in range(2):
        x, u, ids = s.particles(0, sp)
        assert np.array_equal(ids, np.arange(sum(npairs)))
        assert np.abs(G.wrap_delta(x, parts[sp][0], dims)).max() < (1e-12 if fp64 else 2e-6)
        assert G.u_rel_err(u, parts[sp][1], 1e-3).max() < (1e-9 if fp64 else 2e-6)
    d = s.diag(0)
    assert d["flags"] == 0 and d["n_overflow"].tolist() == [0, 0]
    s.step(3)
    assert s.diag(0)["count"].tolist() == [sum(npairs)] * 2
    s.close()


@pytest.mark.parametrize("theta,gb", [(0.02, 0.0), (0.5, 2.0), (8.0, 0.3)])
def test_fp32_momenta_are_the_rounded_fp64_ones(theta, gb):
    # without fields the half step back leaves momenta as they are; the FP64
    # ones are off by roundoff, far below 1e-6 of an FP32 rounding step
    dims, ppc = (16, 16, 16), 64
    u = []
    for fp64 in (False, True):
        s = G.sim(dims, 10.0, 2.0 * ppc, [ppc * 4096] * 2, fp64=fp64)
        s.load(0, 0, 1, (theta, gb, 1), (theta, -gb, 2), ppc, seed=3)
        s.step(0)
        u.append(np.stack([s.particles(0, sp)[1] for sp in range(2)]))
        s.close()
    half = 0.5 * np.spacing(np.abs(u[0]).astype(np.float32)).astype(np.float64)
    assert np.all(np.abs(u[1] - u[0]) <= half * (1.0 + 1e-6))
