"""Spectra of small and of thin boxes: rows on both sides of the lengths that are
read straight from the grid, few modes whose sums are split over the waves of a
block, remainders of the products of four; no trace left in the current."""
import numpy as np
import pytest

from tests import gpu_cases as G
from tests.gpu_trace import trace

pytestmark = pytest.mark.gpu


def _reference(f, dims, axis):
    a = f.reshape(dims[2], dims[1], dims[0])                  # z, y, x
    return (np.abs(np.fft.fft2(np.moveaxis(a, 2 - axis, 0), axes=(1, 2))) ** 2).sum(axis=0)


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("dims", [(1, 1, 256), (1, 64, 3), (8, 63, 2), (9, 65, 1), (31, 66, 3), (32, 67, 2), (2, 3, 1024),
                                  (4, 4, 4), (1, 1, 1)])
def test_spectra_of_small_and_thin_boxes(dims, fp64):
    n = int(np.prod(dims))
    rng = np.random.default_rng(sum(dims))
    e, b = (G.field_storage(rng.standard_normal(3 * n), fp64) for _ in range(2))
    s = G.sim(dims, 10.0, 4.0, [1, 1], dt=0.5, fp64=fp64)
    s.set_fields(0, e, b)
    # b^t = b^{t-dt/2} - (dt/2) curl e^t
    E = e.reshape(3, dims[2], dims[1], dims[0])
    up = lambda c, a: np.roll(E[c], -1, axis=2 - a) - E[c]    # difference along axis a
    curl = np.stack([up(2, 1) - up(1, 2), up(0, 2) - up(2, 0), up(1, 0) - up(0, 1)])
    bt = b.reshape(E.shape) - 0.25 * curl
    # the library forms b^t in the form's precision: three roundings of values below |b| + |curl|
    size = np.abs(b).max() + np.abs(curl).max()
    eps = 2.0 ** -53 if fp64 else 2.0 ** -24
    for axis in range(3):
        for field, comp in ((0, 0), (0, 2), (1, 1)):
            v = (E if field == 0 else bt)[comp].reshape(-1)
            ref = _reference(v, dims, axis)
            got = s.spectrum(0, field, comp, axis)
            # each term of a mode's sum is off by `one` at most, the mode's amplitude by
            # sqrt of the plane's points times as much (random signs; taken six times),
            # and FP64 sums add 1e-14 of the largest
            plane = n // dims[axis]
            one = 4 * eps * size if field else 0.0
            amp = np.sqrt(ref.max())
            tol = 12 * amp * np.sqrt(plane) * one * np.sqrt(dims[axis]) + 1e-12 * ref.max()
            assert np.abs(got - ref).max() <= tol, (axis, field, comp, np.abs(got - ref).max(), tol)
    _, _, j = s.fields(0)
    assert not j.any()
    s.close()


def test_a_small_box_takes_three_kernels():
    s = G.sim((4, 4, 4), 10.0, 4.0, [1, 1])
    for field in range(2):
        s.spectrum(0, field, 0, 0)
        kernels, _, _ = trace(lambda: s.spectrum(0, field, 0, 0))
        assert len(kernels) == 3, kernels
    s.close()
