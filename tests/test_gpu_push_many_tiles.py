"""The push with 256 threads per tile, which contexts of more than 512 tiles
take, against the oracle: a small box with the case, beside a nearly empty box
that brings the tiles.  Packed moves, the hand-over of more leavers than one
batch, the overflow region and its early repack, both solvers."""
import numpy as np
import pytest

from tests import gpu_cases as G
from tests.gpu_trace import trace

pytestmark = pytest.mark.gpu

FILLER = (40, 32, 32)      # 640 tiles


def _sim(dims, n, fp64, **kw):
    from paper_1308_5892_amd import pic as P
    boxes = [{"n": d, "n_x": 10.0, "rho0": 16.0, "max_particles": [m, m]} for d, m in ((dims, n), (FILLER, 50))]
    s = P.Simulation(boxes, G.PAIR, 0.5, fp64=fp64, track_ids=True, **kw)
    rng = np.random.default_rng(1)
    for sp in range(2):
        s.set_particles(1, sp, rng.uniform(0, 1, (50, 3)) * np.array(FILLER), rng.standard_normal((50, 3)))
    st = G.oracle_state(dims, 10.0, 16.0)
    st.faraday4 = bool(kw.get("faraday4"))
    return s, st


def _stepped(s, f4):
    """One step, by the kernel this file is about."""
    kernels, _, _ = trace(lambda: s.step(1))
    push = [k for k in kernels if "push_kernel" in k]
    assert len(push) == 1 and "pic::push_kernel<" in push[0] and f", 1, 0, {int(f4)}>" in push[0], kernels


def _same(s, st, tol, n):
    for sp in range(2):
        x, u, ids = s.particles(0, sp)
        assert np.array_equal(ids, np.arange(n))
        assert G.u_rel_err(u, st.u[st.species == sp], 1e-2).max() < tol
        assert np.abs(G.wrap_delta(x, st.x[st.species == sp], st.dims)).max() < 10 * tol
    e, b, _ = s.fields(0)
    assert np.abs(e - st.e).max() < tol * np.abs(st.e).max()
    assert np.abs(b - st.b).max() < tol * max(np.abs(st.b).max(), np.abs(st.e).max())


# as in the cases with more threads per tile: FP32 roundoff over a few steps,
# and FP64 sums in another order
TOL = {False: 2e-5, True: 1e-11}


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("f4", [False, True], ids=["yee", "fourth_order"])
@pytest.mark.parametrize("dims", [(5, 4, 8), (3, 9, 6), (8, 5, 1), (12, 16, 11)])
def test_packed_moves(dims, f4, fp64):
    rng = np.random.default_rng(sum(dims))
    n = 2600
    s, st = _sim(dims, n, fp64, faraday4=f4)
    e, b = G.random_fields(rng, int(np.prod(dims)), 0.02, 0.2)
    parts = [(rng.uniform(0, 1, (n, 3)) * np.array(dims), 2.0 * rng.standard_normal((n, 3))) for _ in range(2)]
    G.start(s, st, parts, e=e, b=b, fp64=fp64)
    _stepped(s, f4)
    s.step(5)
    st.step(6)
    _same(s, st, TOL[fp64], n)
    assert s.diag(0)["flags"] == 0
    s.close()


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("f4", [False, True], ids=["yee", "fourth_order"])
def test_a_tile_that_bursts(f4, fp64):
    # all particles in one tile of 16, a seventh of which leave it in the first
    # step: more leavers than a block hands over at once (4 x 256), into tiles
    # laid out empty, so that the overflow region (2500 particles per species)
    # takes those beyond the slack
    rng = np.random.default_rng(5)
    dims, n = (16, 8, 8), 4200
    s, st = _sim(dims, 40000, fp64, faraday4=f4, headroom=1.05)
    parts = [(rng.uniform(0, 4, (n, 3)) + np.array([4.0, 4.0, 0.0]), rng.standard_normal((n, 3))) for _ in range(2)]
    G.start(s, st, parts, fp64=fp64)
    x0 = st.x.copy()
    _stepped(s, f4)
    st.step(1)
    left = (np.floor(st.x / 4) != np.floor(x0 / 4)).any(axis=1)
    assert left.sum() > 4 * 256
    seen = int(s.diag(0)["n_overflow"].sum())
    for _ in range(5):
        s.step(1)
        st.step(1)
        seen = max(seen, int(s.diag(0)["n_overflow"].sum()))
    assert seen > 0 and s.diag(0)["flags"] == 0
    _same(s, st, TOL[fp64], n)
    s.close()


@pytest.mark.parametrize("fp64", [False, True])
def test_overflow_watch_repacks_early(fp64):
    # an eighth of the particles stream into tiles laid out empty, with no
    # periodic repack
    from paper_1308_5892_amd import pic as P
    rng = np.random.default_rng(12)
    dims, n = (16, 8, 8), 6000
    s, st = _sim(dims, n, fp64, headroom=1.05, sort_interval=0)
    parts = []
    for _ in range(2):
        u = 0.05 * rng.standard_normal((n, 3))
        u[: n // 8, 0] += 3.0
        parts.append((rng.uniform(0, 1, (n, 3)) * np.array([4.0, 8.0, 8.0]), u))
    G.start(s, st, parts, fp64=fp64)
    P.pic_set_timing(s.ctx, 1)
    _stepped(s, False)
    st.step(1)
    seen = 0
    for _ in range(19):
        s.step(1)
        st.step(1)
        seen = max(seen, int(s.diag(0)["n_overflow"].max()))
    assert seen > 512, seen                  # half the region of 1024
    assert P.pic_get_timing(s.ctx)["sort_launches"] >= 1
    assert s.diag(0)["flags"] == 0
    for sp in range(2):
        x, u, _ = s.particles(0, sp)
        assert len(x) == n
        assert G.u_rel_err(u, st.u[st.species == sp], 1e-3).max() < (1e-11 if fp64 else 1e-5)
    s.close()


def test_runs_with_overflow_are_bitwise_identical():
    def run():
        rng = np.random.default_rng(11)
        dims, n = (16, 8, 8), 4200
        s, st = _sim(dims, 40000, False, headroom=1.05)
        G.start(s, st, [(rng.uniform(0, 4, (n, 3)), rng.standard_normal((n, 3))) for _ in range(2)])
        seen = 0
        for _ in range(8):
            s.step(1)
            seen = max(seen, int(s.diag(0)["n_overflow"].sum()))
        assert s.diag(0)["flags"] == 0
        out = [v for sp in range(2) for v in s.particles(0, sp)] + list(s.fields(0)[:2])
        s.close()
        return out, seen

    (a, seen), (b, _) = run(), run()
    assert seen > 0
    assert all(np.array_equal(x, y) for x, y in zip(a, b))
