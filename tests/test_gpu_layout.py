"""The segment layout of a repack at the edges of its blocks: tile counts around
256 and 1024, one pass and several, boxes of many and of few tiles together.  An
FP32 run does not depend on the layout, so a run that repacks at every step
equals one that never does, bit for bit."""
import numpy as np
import pytest

from tests import gpu_cases as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("boxes", [[(255, 1, 1)], [(256, 1, 1)], [(257, 1, 1)], [(1023, 1, 1)], [(1024, 1, 1)], [(41, 25, 1)],
                                   [(2048, 1, 1)], [(683, 3, 1)], [(2, 1, 1), (1, 1, 1), (700, 1, 1), (3, 2, 1)],
                                   [(600, 2, 1), (1, 1, 1), (1500, 1, 1)]],
                         ids=lambda b: "+".join(str(int(np.prod(d))) for d in b))
def test_repacks_change_nothing(boxes):
    from paper_1308_5892_amd import pic as P

    def run(sort_interval):
        rng = np.random.default_rng(len(boxes))
        n = 1500
        s = P.Simulation([{"n": d, "n_x": 10.0, "rho0": 8.0, "max_particles": [n, n], "tile": (1, 1, 1)} for d in boxes],
                         G.PAIR, 0.5, track_ids=True, sort_interval=sort_interval)
        for b, d in enumerate(boxes):
            for sp in range(2):
                x = rng.uniform(0, 1, (n, 3)) * np.array(d)
                s.set_particles(b, sp, x, 0.5 * rng.standard_normal((n, 3)))
        s.step(4)
        out = []
        for b in range(len(boxes)):
            d = s.diag(b)
            assert d["flags"] == 0 and d["count"].tolist() == [n, n]
            for sp in range(2):
                x, u, ids = s.particles(b, sp)
                assert np.array_equal(ids, np.arange(n))
                out += [x, u]
            out += list(s.fields(b)[:2])
        s.close()
        return out

    assert all(np.array_equal(a, b) for a, b in zip(run(0), run(1)))
