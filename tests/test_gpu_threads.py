"""Several threads: boxes of one context copied to and from the host at the same
time, and contexts loaded at the same time (the library's calls release
Python's lock)."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from tests import gpu_cases as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp64", [False, True])
def test_boxes_of_one_context_copied_by_several_threads(fp64):
    # boxes whose fields are read at once and in parts, and different numbers of
    # particles; each thread has a box and checks every value it gets
    from paper_1308_5892_amd import pic as P
    dims = [(4, 4, 4), (16, 16, 16), (9, 7, 5), (30, 20, 25), (8, 8, 8), (24, 24, 24)]
    rng = np.random.default_rng(3)
    n = [200 * (k + 1) for k in range(len(dims))]
    s = P.Simulation([{"n": d, "n_x": 10.0, "rho0": 8.0, "max_particles": [m, m]} for d, m in zip(dims, n)], G.PAIR, 0.5,
                     fp64=fp64, track_ids=True)
    want = []
    for b, (d, m) in enumerate(zip(dims, n)):
        c = 3 * int(np.prod(d))
        x, u = G.to_storage(rng.uniform(0, 1, (m, 3)) * np.array(d), rng.standard_normal((m, 3)), d, fp64)
        want.append((G.field_storage(rng.standard_normal(c), fp64), G.field_storage(rng.standard_normal(c), fp64), x, u))
        s.set_fields(b, *want[b][:2])
        for sp in range(2):
            s.set_particles(b, sp, x, u)
    s.step(0)                                    # binned: the copies below change nothing

    def work(b):
        e, f, x, u = want[b]
        for k in range(25):
            got = s.fields(b)
            assert np.array_equal(got[0], e) and np.array_equal(got[1], f) and not got[2].any(), (b, k)
            gx, gu, ids = s.particles(b, k % 2)
            assert np.array_equal(ids, np.arange(n[b])) and np.array_equal(gx, x) and np.array_equal(gu, u), (b, k)
            s.set_fields(b, e, f if k % 3 else None)
        return b

    with ThreadPoolExecutor(len(dims)) as pool:
        assert list(pool.map(work, range(len(dims)))) == list(range(len(dims)))
    s.close()


def test_contexts_loaded_by_several_threads():
    # tile shapes whose backward half step needs different amounts of LDS, all
    # above the default limit of 64 KiB; a load's momenta depend on nothing else
    import torch
    from paper_1308_5892_amd import pic as P
    tiles = [(8, 4, 4), (8, 8, 4), (4, 8, 8), (8, 8, 2)]
    dims, ppc = (16, 16, 8), 2
    n = ppc * int(np.prod(dims))
    rng = np.random.default_rng(2)
    e, b = G.random_fields(rng, int(np.prod(dims)), 0.02, 0.2)

    def load(tile):
        with torch.cuda.stream(torch.cuda.Stream()):
            out = []
            for _ in range(6):
                s = P.Simulation([{"n": dims, "n_x": 10.0, "rho0": 4.0, "max_particles": [n, n], "tile": tile}], G.PAIR, 0.5,
                                 fp64=True, track_ids=True)
                s.set_fields(0, e, b)
                s.load(0, 0, 1, (0.2, 0.3, 0), (0.2, -0.3, 0), ppc, seed=4)
                s.step(0)
                out.append(s.particles(0, 0)[1])
                s.step(2)
                s.sync()
                s.close()
            return out

    ref = load(tiles[0])[0]
    with ThreadPoolExecutor(len(tiles)) as pool:
        for got in pool.map(load, tiles):
            assert all(np.array_equal(u, got[0]) for u in got)
            assert np.abs(got[0] - ref).max() <= 1e-13 * np.abs(ref).max()    # the same sums, in FP64
