"""The diagnostics' shortcuts: histogram bins decided by an FP32 logarithm, sums
held over several tiles per block, boxes of more tiles than blocks."""
import numpy as np
import pytest

from tests import gpu_cases as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("bins,lo,hi", [(7, -3.0, 1.5), (512, -4.0, 3.0), (513, -1.0, 0.0), (60000, -2.0, 2.0)])
def test_histogram_counts_are_those_of_the_fp64_logarithm(bins, lo, hi, fp64):
    # without fields u^- is u, so the read-back particles give every bin; a
    # value within roundoff of an edge may fall on either side
    rng = np.random.default_rng(bins)
    dims, n = (6, 5, 4), 20000
    s = G.sim(dims, 10.0, 16.0, [n, n], fp64=fp64, hist_bins=bins, hist_lo=lo, hist_hi=hi)
    for sp in range(2):
        u = rng.standard_normal((n, 3)) * 10.0 ** rng.uniform(-3, 1.2, (n, 1))
        u[:50] = 0.0                                     # gamma - 1 = 0: the lowest bin
        s.set_particles(0, sp, rng.uniform(0, 1, (n, 3)) * np.array(dims), u)
    got = s.diag(0, hist_bins=bins)["hist"]
    for sp in range(2):
        _, u, _ = s.particles(0, sp)
        g = np.sqrt(1.0 + u[:, 0] ** 2 + u[:, 1] ** 2 + u[:, 2] ** 2) - 1.0
        x = (np.log10(np.maximum(g, 1e-300)) - lo) / (hi - lo) * bins
        ref = np.bincount(np.clip(np.floor(x), 0, bins - 1).astype(int), minlength=bins)
        # roundoff of gamma - 1 (2^-52 of gamma) and of the logarithm, in bins
        err = (4e-16 * (1.0 + g) / np.maximum(g, 1e-16) + 1e-14) * bins / (hi - lo)
        near = int(np.sum(np.abs(x - np.round(x)) < err))
        assert got[sp].sum() == n
        assert np.abs(got[sp] - ref).sum() <= 2 * near, (np.abs(got[sp] - ref).sum(), near)
    s.close()


@pytest.mark.parametrize("fp64", [False, True])
def test_sums_over_more_tiles_than_blocks(fp64):
    # 2176 tiles, most of them empty, and particles in the others
    rng = np.random.default_rng(8)
    dims, n = (34, 32, 16), 3000
    s = G.sim(dims, 10.0, 16.0, [n, n], fp64=fp64, tile=(2, 2, 2))
    st = G.oracle_state(dims, 10.0, 16.0)
    e, b = G.random_fields(rng, int(np.prod(dims)), 0.02, 0.2)
    parts = [(rng.uniform(0, 1, (n, 3)) * np.array([34.0, 8.0, 5.0]), rng.standard_normal((n, 3))) for _ in range(2)]
    G.start(s, st, parts, e=e, b=b, fp64=fp64)
    d, ref = s.diag(0), st.diag()
    rel = 1e-10 if fp64 else 1e-5
    assert d["count"].tolist() == [n, n] and d["flags"] == 0
    for k in ("W_E", "W_B", "K"):
        assert np.all(np.abs(d[k] - ref[k]) <= rel * np.abs(ref[k])), (k, d[k], ref[k])
    assert abs(d["gauss_max"] - ref["gauss_max"]) <= rel * ref["gauss_max"]
    s.close()
