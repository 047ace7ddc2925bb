"""The Gauss residual of fields that hold NaN: a box without particles, whose
residual is div e, against numpy on the values as stored."""
import ctypes as C

import numpy as np
import pytest

from tests import gpu_cases as G

pytestmark = pytest.mark.gpu

DIMS = (64, 3, 2)      # a row along x is one wave's 64 nodes


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("filt", [False, True], ids=["plain", "smoothed"])
@pytest.mark.parametrize("bad", ["none", "one", "63_of_a_wave", "wave", "component", "all"])
def test_gauss_max_of_fields_with_nan(bad, filt, fp64):
    from paper_1308_5892_amd import pic as P
    rng = np.random.default_rng(5)
    n = int(np.prod(DIMS))
    e = G.field_storage(rng.standard_normal(3 * n), fp64).reshape(3, DIMS[2], DIMS[1], DIMS[0])
    if bad == "one":
        e[0, 1, 1, 7] = np.nan
    elif bad == "63_of_a_wave":
        e[0, 1, 1, :62] = np.nan                 # the residual of nodes 0..62 of the row
    elif bad == "wave":
        e[0, 1, 1] = np.nan
    elif bad == "component":
        e[2] = np.nan
    elif bad == "all":
        e[:] = np.nan
    div = sum(e[c] - np.roll(e[c], 1, axis=2 - c) for c in range(3))
    waves = np.abs(div).reshape(-1, 64)
    # per wave the largest residual that is a number, NaN if none is; any NaN of these wins
    per = [np.nan if np.isnan(w).all() else np.nanmax(w) for w in waves]
    ref = np.nan if np.isnan(per).any() else max(per)
    s = G.sim(DIMS, 10.0, 4.0, [1, 1], fp64=fp64, filter_current=filt)
    s.set_fields(0, e.reshape(-1), np.zeros(3 * n))
    for call in ("pic_diag", "pic_diag_noalloc"):
        d = P.pic_diag_out()
        assert getattr(P.lib(), call)(s.ctx, 0, C.byref(d), None) == P.PIC_OK
        # FP64 differences of the stored values in another order: a few ulp of the terms
        assert np.isclose(d.gauss_max, ref, rtol=1e-13, atol=1e-13, equal_nan=True), (call, d.gauss_max, ref)
        assert np.isnan(d.gauss_rms) == np.isnan(div).any()
    s.close()
