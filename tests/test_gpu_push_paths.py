"""The push's 4x4x4-tile loop against the oracle where its packed cell words can
go wrong: full tiles, partial tiles at the box's far end and the moves down
into them, two tiles per axis, and axes that one tile spans."""
import numpy as np
import pytest

from tests import gpu_cases as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("dims", [(4, 4, 4), (5, 4, 8), (3, 9, 6), (2, 13, 7), (8, 5, 1), (12, 16, 11)])
def test_packed_moves(dims, fp64):
    # hot particles (most moves cross a face) over enough steps that every
    # tile hands particles to every neighbour; tolerances as for the other
    # few-step runs against the oracle, scaled to the steps
    rng = np.random.default_rng(sum(dims))
    n = 2600
    s = G.sim(dims, 10.0, 40.0, [n, n], fp64=fp64)
    st = G.oracle_state(dims, 10.0, 40.0)
    e, b = G.random_fields(rng, int(np.prod(dims)), 0.02, 0.2)
    parts = [(rng.uniform(0, 1, (n, 3)) * np.array(dims), 2.0 * rng.standard_normal((n, 3))) for _ in range(2)]
    G.start(s, st, parts, e=e, b=b, fp64=fp64)
    s.step(6)
    st.step(6)
    tol = 1e-11 if fp64 else 2e-5
    for sp in range(2):
        x, u, ids = s.particles(0, sp)
        assert np.array_equal(ids, np.arange(n))
        assert np.all((x >= 0) & (x < np.array(dims, float)))
        assert G.u_rel_err(u, st.u[st.species == sp], 1e-2).max() < tol
        assert np.abs(G.wrap_delta(x, st.x[st.species == sp], dims)).max() < 10 * tol
    e1, b1, _ = s.fields(0)
    assert np.abs(e1 - st.e).max() < tol * np.abs(st.e).max()
    assert np.abs(b1 - st.b).max() < tol * np.abs(st.b).max()
    assert s.diag(0)["flags"] == 0
    s.close()


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("kw", [{}, {"faraday4": True}, {"tile": (8, 4, 2)}], ids=["yee", "fourth_order", "tile842"])
def test_particles_enter_empty_tiles(fp64, kw):
    # all particles start in one corner tile of a box with an evolving field:
    # the empty tiles still advance b, and take the particles that enter them
    # without the overflow region (each tile has 32 slots to spare, and fewer
    # than that enter any of them here)
    rng = np.random.default_rng(77)
    dims, n = (17, 12, 8), 40
    s = G.sim(dims, 10.0, 40.0, [n, n], fp64=fp64, **kw)
    st = G.oracle_state(dims, 10.0, 40.0)
    st.faraday4 = bool(kw.get("faraday4"))
    e, b = G.random_fields(rng, int(np.prod(dims)), 0.02, 0.2)
    parts = [(rng.uniform(0, 3, (n, 3)), rng.standard_normal((n, 3))) for _ in range(2)]
    G.start(s, st, parts, e=e, b=b, fp64=fp64)
    tol = 1e-11 if fp64 else 2e-5
    for _ in range(3):
        s.step(4)
        st.step(4)
        e1, b1, _ = s.fields(0)
        assert np.abs(e1 - st.e).max() < tol * np.abs(st.e).max()
        assert np.abs(b1 - st.b).max() < tol * np.abs(st.b).max()
        d = s.diag(0)
        assert d["flags"] == 0 and d["count"].tolist() == [n, n] and d["n_overflow"].tolist() == [0, 0]
    for sp in range(2):
        x, u, _ = s.particles(0, sp)
        assert np.abs(G.wrap_delta(x, st.x[st.species == sp], dims)).max() < 10 * tol
        assert G.u_rel_err(u, st.u[st.species == sp], 1e-2).max() < 10 * tol
    s.close()


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("dims", [(24, 24, 28), (32, 24, 32), (32, 36, 29)], ids=["252_tiles", "384_tiles", "576_tiles"])
def test_block_sizes(dims, fp64):
    # one tile per CU, two, and more: the push with 1024 (FP32), 512 and 256
    # threads per tile against the oracle, at a density that gives a wave none to
    # several particles of a tile
    rng = np.random.default_rng(dims[2])
    n = 12000
    s = G.sim(dims, 10.0, 16.0, [n, n], fp64=fp64)
    st = G.oracle_state(dims, 10.0, 16.0)
    e, b = G.random_fields(rng, int(np.prod(dims)), 0.02, 0.2)
    side = np.array(dims) / np.array([1.0, 6.0, 1.0])        # a dense slab, the rest empty
    parts = [(rng.uniform(0, 1, (n, 3)) * side, 0.7 * rng.standard_normal((n, 3))) for _ in range(2)]
    G.start(s, st, parts, e=e, b=b, fp64=fp64)
    s.step(4)
    st.step(4)
    tol = 1e-11 if fp64 else 2e-5
    for sp in range(2):
        x, u, ids = s.particles(0, sp)
        assert np.array_equal(ids, np.arange(n))
        assert G.u_rel_err(u, st.u[st.species == sp], 1e-2).max() < tol
        assert np.abs(G.wrap_delta(x, st.x[st.species == sp], dims)).max() < 10 * tol
    e1, b1, _ = s.fields(0)
    assert np.abs(e1 - st.e).max() < tol * np.abs(st.e).max()
    assert np.abs(b1 - st.b).max() < tol * np.abs(st.b).max()
    assert s.diag(0)["flags"] == 0
    s.close()
