"""Plane spectra against numpy's FFT at the edges of the matrix tiles: fewer
and more than 16 modes, odd sizes, one plane and many, one cell along an axis."""
import numpy as np
import pytest

from tests import gpu_cases as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("dims", [(1, 1, 1), (2, 1, 3), (17, 16, 15), (33, 5, 64), (130, 31, 1), (1, 3, 257), (32, 300, 2)])
def test_spectra_of_e_match_an_fft(dims, fp64):
    rng = np.random.default_rng(sum(dims))
    cells = int(np.prod(dims))
    s = G.sim(dims, 10.0, 16.0, [1, 1], fp64=fp64)
    e = G.field_storage(rng.standard_normal(3 * cells), fp64)
    s.set_fields(0, e, np.zeros(3 * cells))
    for comp in range(3):
        f = e[comp * cells:(comp + 1) * cells].reshape(dims[2], dims[1], dims[0])
        for normal in range(3):
            ax = tuple(2 - a for a in range(3) if a != normal)
            ref = (np.abs(np.fft.fftn(f, axes=ax)) ** 2).sum(2 - normal)
            got = s.spectrum(0, 0, comp, normal)
            # FP64 sums of N1 N2 terms and of the planes' powers
            assert got.shape == ref.shape
            assert np.abs(got - ref).max() <= 1e-12 * ref.max(), (comp, normal)
    # the scratch is cleared: a vacuum step sees no current
    s.set_fields(0, np.zeros(3 * cells), np.zeros(3 * cells))
    s.spectrum(0, 1, 0, 2)
    s.step(1)
    e1, b1, j1 = s.fields(0)
    assert not e1.any() and not b1.any() and not j1.any()
    s.close()
