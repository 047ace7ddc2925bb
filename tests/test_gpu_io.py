"""Host copies: values as given, order by id for ids of any kind, outputs larger
than one pass of the conversion, and no trace left in the next step."""
import numpy as np
import pytest

from tests import gpu_cases as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("ids", ["permuted", "offset", "repeated", "negative"])
def test_particles_come_back_ordered_by_id(ids, fp64):
    rng = np.random.default_rng(31)
    dims, n = (9, 7, 5), 5000                    # 5000 of a capacity of 5000: several passes in the FP32 form
    s = G.sim(dims, 10.0, 16.0, [n, n], fp64=fp64)
    x = rng.uniform(-1, 2, (n, 3)) * np.array(dims)          # wrapped into the box
    u = rng.standard_normal((n, 3))
    given = {"permuted": rng.permutation(n), "offset": 100 + rng.permutation(n), "repeated": rng.permutation(n) // 2,
             "negative": rng.permutation(n) - 7}[ids].astype(np.int32)
    s.set_particles(0, 0, x, u, given)
    s.set_particles(0, 1, x[:0], u[:0])
    gx, gu, gi = s.particles(0, 0)
    order = np.argsort(given, kind="stable")
    xs, us = G.to_storage(x, u, dims, fp64)
    assert np.array_equal(gi, given[order])
    if ids == "repeated":                                    # equal ids in either order
        gx, gu = [np.sort(v.reshape(n // 2, 2, 3), axis=1) for v in (gx, gu)]
        xs, us = [np.sort(v[order].reshape(n // 2, 2, 3), axis=1) for v in (xs, us)]
    else:
        xs, us = xs[order], us[order]
    assert np.array_equal(gx, xs) and np.array_equal(gu, us)
    assert len(s.particles(0, 1)[0]) == 0
    s.close()


@pytest.mark.parametrize("fp64", [False, True])
def test_particles_without_ids_come_back_once_each(fp64):
    from paper_1308_5892_amd import pic as P
    rng = np.random.default_rng(32)
    dims, n = (8, 12, 6), 4000
    s = P.Simulation([{"n": dims, "n_x": 10.0, "rho0": 16.0, "max_particles": [n, n]}], G.PAIR, 0.5, fp64=fp64)
    x, u = rng.uniform(0, 1, (n, 3)) * np.array(dims), rng.standard_normal((n, 3))
    s.set_particles(0, 0, x, u)
    s.set_particles(0, 1, x, u)
    xs, us = G.to_storage(x, u, dims, fp64)
    for sp in range(2):
        gx, gu, gi = s.particles(0, sp)
        assert len(gx) == n and not gi.any()
        a, b = np.concatenate([gx, gu], 1), np.concatenate([xs, us], 1)
        assert np.array_equal(a[np.lexsort(a.T)], b[np.lexsort(b.T)])
    with pytest.raises(P.PicError) as ei:
        P.pic_get_particles(s.ctx, 0, 0, n - 1)
    assert ei.value.code == P.PIC_ENOMEM
    s.close()


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("wall", [0, 1, 2, 3])
def test_fields_come_back_as_stored_and_leave_no_current(wall, fp64):
    from paper_1308_5892_amd import pic as P
    rng = np.random.default_rng(33)
    dims = (7, 5, 6)
    cells = int(np.prod(dims))
    s = P.Simulation([{"n": dims, "n_x": 10.0, "rho0": 16.0, "max_particles": [1, 1], "walls": wall}], G.PAIR, 0.5,
                     fp64=fp64)
    e, b = rng.standard_normal(3 * cells), rng.standard_normal(3 * cells)
    s.set_fields(0, e, None)
    s.set_fields(0, None, b)
    re, rb = [G.field_storage(v, fp64).reshape(3, dims[2], dims[1], dims[0]) for v in (e, b)]
    if wall:
        for c in range(3):
            (rb if c == wall - 1 else re)[c].swapaxes(0, 3 - wall)[0] = 0.0
    for _ in range(2):
        ge, gb, gj = s.fields(0)
        assert np.array_equal(ge, re.reshape(-1)) and np.array_equal(gb, rb.reshape(-1)) and not gj.any()
    s.set_fields(0, np.zeros(3 * cells), np.zeros(3 * cells))
    s.step(1)
    ge, gb, _ = s.fields(0)
    assert not ge.any() and not gb.any()
    s.close()


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("dims", [(16, 16, 34), (32, 22, 31), (31, 30, 47)], ids=["one_part", "just_over", "parts_and_rest"])
def test_fields_come_back_in_parts(dims, fp64):
    # parts of 65536 FP32 or 32768 FP64 values: 26112, 65472 and 131130 values
    # per field; what a field holds comes back exactly, and reading it changes
    # nothing (the second read)
    n = int(np.prod(dims))
    rng = np.random.default_rng(n)
    e, b = (rng.standard_normal(3 * n).astype(np.float32).astype(np.float64) for _ in range(2))
    s = G.sim(dims, 10.0, 2.0, [64, 64], fp64=fp64)
    s.set_fields(0, e, b)
    for _ in range(2):
        e1, b1, j1 = s.fields(0)
        assert np.array_equal(np.ravel(e1), e) and np.array_equal(np.ravel(b1), b) and not np.any(j1)
    s.close()
