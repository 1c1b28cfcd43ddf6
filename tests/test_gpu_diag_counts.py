"""The instability counts and the general caloric law in every kernel of the
statistics: nodes that are not finite or not positive at the edges of tiles and
in the last plane of a chunk are counted once each, and C_v(T) enters the energy
and the speed of sound with a moving reference state."""
import numpy as np
import pytest

from paper_2102_09512_amd import inputs as I
from test_diag_geometry_rule import _grid
from test_gpu_field_paths import _sums

pytestmark = pytest.mark.gpu

# marching over 128 x 1, 32 x 8, 64 x 8 and 32 x 16 tiles, and memory order in both lattices
BOXES = [(2, (300, 90)), (2, (20, 300)), (3, (40, 30, 12)), (3, (100, 90, 80)), (3, (88, 92, 139)), (3, (5, 30, 20))]


def _edges(dims, g):
    """Nodes at the box's corners and, where it is marched in tiles, on both sides of a tile's edges in the planes
    around the end of a chunk."""
    x, y, z = (*dims, *[1] * (3 - len(dims)))
    at = {(0, 0, 0), (x - 1, y - 1, z - 1), (x // 2, 0, z - 1)}
    if not g.flat:
        m = (z if len(dims) == 3 else y) - 1
        for p in {min(g.chunk - 1, m), min(g.chunk, m)}:
            for tx in {min(g.bx - 1, x - 1), min(g.bx, x - 1)}:
                if len(dims) == 2:
                    at.add((tx, p, 0))
                else:
                    at |= {(tx, min(g.by - 1, y - 1), p), (tx, min(g.by, y - 1), p)}
    return sorted(a + x * (b + y * c) for a, b, c in at)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("lattice,dims", BOXES)
def test_every_bad_node_is_counted_once(lattice, dims, precision):
    from paper_2102_09512_amd import lbm

    print("[gpu case] instability counts", lattice, dims, precision, flush=True)
    g, N, Q = _grid(dims, precision), int(np.prod(dims)), 9 if lattice == 2 else 27
    nodes = _edges(dims, g)
    h = lbm.lbm_create(lattice, dims, 1.4, 0.7, 0.02, precision=precision, T_ref=0.15)
    try:
        lbm.lbm_init_fields(h, *I.smooth_random(lattice, dims, seed=4))
        good = np.empty((2, Q, N), dtype=np.float64 if precision == 0 else np.float32)
        lbm.lbm_get_state(h, good)
        # plane, value: g of a node that is not a number, f that is infinite, a negative density, a negative energy
        for plane, value, key in ((Q, np.nan, "nonfinite"), (0, np.inf, "nonfinite"), (0, -10.0, "nonpositive"),
                                  (Q, -10.0, "nonpositive")):
            for some in (nodes[:1], nodes[-1:], nodes):
                s = good.copy()
                s.reshape(2 * Q, N)[plane, some] = value
                lbm.lbm_set_state(h, s)
                for call in (lbm.lbm_diagnostics, lbm.lbm_diagnostics_noalloc):
                    d = call(h)
                    assert d[key] == len(some) and d["nodes"] == N, (key, some)
                    if value == -10.0:
                        assert d["nonfinite"] == 0
                with pytest.raises(lbm.LbmError) as e:
                    lbm.lbm_step(h, 1)
                assert e.value.code == lbm.LBM_EUNSTABLE
        lbm.lbm_set_state(h, good)
        d = lbm.lbm_diagnostics(h)
        assert d["nonfinite"] == d["nonpositive"] == 0
    finally:
        lbm.lbm_destroy(h)


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("lattice,dims", BOXES)
def test_general_caloric_law_with_a_moving_reference(lattice, dims, precision):
    from paper_2102_09512_amd import lbm

    c = (2.5, 0.4, 0.2)
    print("[gpu case] caloric statistics", lattice, dims, precision, flush=True)
    rho, u, T = I.smooth_random(lattice, dims, seed=5)
    u = u + 0.03
    h = lbm.lbm_create(lattice, dims, 1.4, 0.7, 0.02, precision=precision, T_ref=0.15, visc_exponent=0.76, bc=(1, 0, 0),
                       u_ref=(0.1, -0.05, 0.02)[:lattice], cv_poly=c)
    try:
        lbm.lbm_init_fields(h, rho, u, T)
        m = [np.empty_like(a) for a in (rho, u, T)]
        lbm.lbm_moments(h, *m)
        got = lbm.lbm_diagnostics(h)
        assert got == lbm.lbm_diagnostics_noalloc(h)
        # the coefficients as stored: rounded to FP32 with FP32 storage
        c0, c1, c2 = (np.float32(k).astype(np.float64) if precision else k for k in c)
        ref = _sums(lattice, *m, [True, False, False], 0.02, 0.76, 0.15, 2.5)
        cv = c0 + c1 * m[2] + c2 * m[2] ** 2
        ref["cs_sum"] = np.sqrt((cv + 1) / cv * m[2]).sum()
        U = c0 * m[2] + c1 * m[2] ** 2 / 2 + c2 * m[2] ** 3 / 3
        ref["energy"] = (m[0] * (U + 0.5 * (m[1] ** 2).sum(0))).sum()
        for k, v in ref.items():
            # as for the constant law: a few thousand roundings of relative size 2^-53; Newton's T is good to 1e-15
            scale = np.abs(np.asarray(v)) + 1e-10 * rho.size
            assert np.all(np.abs(np.asarray(got[k]) - np.asarray(v)) <= 1e-11 * scale), (k, got[k], v)
    finally:
        lbm.lbm_destroy(h)
