"""What the field copies move: a single field of a box does not take the others
along, and every combination of fields comes back as stored."""
import numpy as np
import pytest

from tests import gpu_cases as G
from tests.gpu_trace import trace

pytestmark = pytest.mark.gpu


def _get(s, n, want):
    from paper_1308_5892_amd import pic as P
    out = [np.full(3 * n, 7.0) if w else None for w in want]
    P._check(P.lib().pic_get_fields(s.ctx, 0, *[P._ptr(a) for a in out]), s.ctx)
    return out


# FP32 boxes read in one copy (all fields within 512 KiB) with single fields
# below and above 16 KiB, and one read in parts
@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("dims", [(1, 1, 1), (11, 11, 11), (19, 18, 4), (16, 16, 33), (30, 31, 33)])
def test_any_combination_of_fields(dims, fp64):
    n = int(np.prod(dims))
    rng = np.random.default_rng(n)
    e, b = (G.field_storage(rng.standard_normal(3 * n), fp64) for _ in range(2))
    s = G.sim(dims, 10.0, 2.0, [1, 1], fp64=fp64)
    for steps in (0, 1):                      # a step swaps the two buffers of b
        s.step(steps)
        s.set_fields(0, e, b)
        for want in np.ndindex(2, 2, 2):
            got = _get(s, n, want)
            for a, ref in zip(got, (e, b, np.zeros(3 * n))):
                assert a is None or np.array_equal(a, ref), (want, steps)
    s.close()


@pytest.mark.parametrize("fp64", [False, True])
def test_one_field_moves_alone(fp64):
    dims = (16, 16, 16) if fp64 else (16, 16, 33)
    n, size = int(np.prod(dims)), 8 if fp64 else 4
    s = G.sim(dims, 10.0, 2.0, [1, 1], fp64=fp64)
    s.step(1)
    s.sync()
    for want, value in (((1, 0, 0), size), ((0, 1, 0), size), ((0, 0, 1), 8)):
        _, to_host, _ = trace(lambda: _get(s, n, want))
        assert to_host == 3 * n * value, want
    s.close()


# both ways through the parts' edges: in values per field, 98304 = three FP64
# read parts, 65538 = one FP32 read part and two values, 131070 and 65535 = the
# last boxes set through the buffer as a whole (FP32, FP64), 131076 the first in
# parts, 393216 = six full parts
@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("dims", [(32, 32, 32), (66, 331, 1), (10, 17, 257), (5, 17, 257), (12, 11, 331), (64, 32, 64)],
                         ids=lambda d: str(3 * int(np.prod(d))))
def test_fields_of_boxes_at_the_edges_of_parts(dims, fp64):
    n = int(np.prod(dims))
    rng = np.random.default_rng(n)
    e, b = (G.field_storage(rng.standard_normal(3 * n), fp64) for _ in range(2))
    s = G.sim(dims, 10.0, 2.0, [1, 1], fp64=fp64)
    for given in ((e, b), (None, -e), (2 * b, None)):
        s.set_fields(0, *given)
        ref = [new if new is not None else old for new, old in zip(given, (e, -e))]
        got_e, got_b, got_j = s.fields(0)
        assert np.array_equal(got_e, ref[0]) and np.array_equal(got_b, ref[1]) and not got_j.any()
    s.close()


@pytest.mark.parametrize("fp64", [False, True])
@pytest.mark.parametrize("dims", [(16, 16, 16), (36, 36, 36)], ids=["at_once", "larger"])
def test_set_fields_moves_what_the_form_stores(dims, fp64):
    n = int(np.prod(dims))
    s = G.sim(dims, 10.0, 2.0, [1, 1], fp64=fp64)
    f = np.ones(3 * n)
    kernels, _, to_device = trace(lambda: s.set_fields(0, f, f))
    assert to_device == 2 * 3 * n * (8 if fp64 else 4) and not kernels
    s.close()
