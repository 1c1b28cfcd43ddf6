"""The statistics in every tile shape and geometry that they are launched in:
edges of the tiles, ragged boxes, work-group counts that eight dies do not share
evenly, and more tiles than work-groups, against plain numpy sums."""
import numpy as np
import pytest

from paper_2102_09512_amd import inputs as I
from test_diag_geometry_rule import _grid
from test_gpu_field_paths import _sums

pytestmark = pytest.mark.gpu

# (lattice, dims, tile or None for memory order, more tiles than work-groups)
CASES = [
    (3, (32, 8, 1), (32, 8), False), (3, (47, 9, 30), (32, 8), False), (3, (31, 7, 250), (32, 8), False),
    (3, (20, 100, 100), (32, 8), False), (3, (64, 64, 64), (32, 8), False), (3, (65, 65, 64), (32, 8), False),
    (3, (64, 8, 600), (64, 8), False), (3, (97, 33, 101), (64, 8), False), (3, (100, 90, 80), (64, 8), False),
    (3, (88, 92, 139), (32, 16), False), (3, (129, 63, 41), (32, 16), False),
    (3, (1100, 1000, 2), (64, 8), True), (2, (262273, 2), (128, 1), True),
]


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("bc", [(0, 0, 0), (1, 0, 1), (0, 1, 0)])
@pytest.mark.parametrize("lattice,dims,tile,more", CASES)
def test_sums(lattice, dims, tile, more, bc, precision):
    from paper_2102_09512_amd import lbm

    print("[gpu case] statistics", lattice, dims, bc, precision, flush=True)
    g = _grid(dims, precision)
    assert not g.flat and (g.bx, g.by) == tile and (g.tasks > g.blocks) == more
    rho, u, T = I.smooth_random(lattice, dims, seed=5)
    u = u + 0.03
    h = lbm.lbm_create(lattice, dims, 1.4, 0.7, 0.02, precision=precision, bc=bc, visc_exponent=0.76, T_ref=0.15)
    try:
        lbm.lbm_init_fields(h, rho, u, T)
        m = [np.empty_like(a) for a in (rho, u, T)]
        lbm.lbm_moments(h, *m)
        got = lbm.lbm_diagnostics(h)
        assert got == lbm.lbm_diagnostics_noalloc(h) == lbm.lbm_diagnostics(h)
        for k, v in _sums(lattice, *m, [b == 1 for b in bc], 0.02, 0.76, 0.15, 2.5).items():
            # a few thousand roundings of relative size 2^-53, on sums whose terms have one sign or a mean
            # velocity well above their scatter; the differences lose |u| / |du| <= 1e3 more
            scale = np.abs(np.asarray(v)) + 1e-10 * rho.size
            assert np.all(np.abs(np.asarray(got[k]) - np.asarray(v)) <= 1e-11 * scale), (k, got[k], v)
        assert got["nonfinite"] == got["nonpositive"] == 0
    finally:
        lbm.lbm_destroy(h)
