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
