"""A launch shape given with chunk 0 gets the default chunk for that shape: where
it is the shape that the box has by default, the whole default tile."""
import numpy as np
import pytest

from paper_2102_09512_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("lattice,dims", [(2, (800, 4)), (2, (300, 300)), (2, (1100, 40)), (3, (20, 25, 40)),
                                          (3, (64, 64, 64)), (3, (100, 50, 61)), (3, (99, 105, 100))])
def test_the_default_shape_given_is_the_default(lattice, dims, precision):
    from paper_2102_09512_amd import lbm

    print("[gpu case] shape without a chunk", lattice, dims, precision, flush=True)

    def tile(t):
        h = lbm.lbm_create(lattice, dims, 1.4, 0.7, 0.02, precision=precision, T_ref=0.15, tile=t)
        try:
            return lbm.lbm_get_tile(h)
        finally:
            lbm.lbm_destroy(h)

    own = tile(None)
    assert tile((own[0], own[1], 0)) == own
    assert tile((own[0], 0, 0)) == own


def test_another_shape_has_a_chunk_and_the_same_results():
    from paper_2102_09512_amd import lbm

    dims = (40, 24, 30)
    print("[gpu case] both FP64 shapes without a chunk", dims, flush=True)
    f, out = I.smooth_random(3, dims, seed=8), []
    for t in (None, (64, 4, 0), (32, 8, 0)):
        h = lbm.lbm_create(3, dims, 1.4, 0.7, 0.02, T_ref=0.15, tile=t)
        try:
            assert 1 <= lbm.lbm_get_tile(h)[2] <= dims[2]
            lbm.lbm_init_fields(h, *f)
            lbm.lbm_step(h, 4)
            m = [np.empty_like(a) for a in f]
            lbm.lbm_moments(h, *m)
            out.append(m)
        finally:
            lbm.lbm_destroy(h)
    for m in out[1:]:
        for a, b in zip(m, out[0]):
            assert np.abs(a - b).max() <= 1e-13  # values up to 1, four steps of FP64 rounding
