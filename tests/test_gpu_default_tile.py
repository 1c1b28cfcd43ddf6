"""The default launch shape at sizes where it changes: whatever march chunk it
takes, the state is that of any other chunk of the shape, bit for bit (FP64,
and the one 512-thread FP32 shape: one plane in flight, one copy of a plane's
arithmetic)."""
import numpy as np
import pytest

from paper_2102_09512_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lattice,dims,precision", [
    (2, (1, 1), 0), (2, (800, 4), 0), (2, (129, 33), 0), (2, (300, 300), 0), (2, (1025, 70), 0),
    (3, (1, 1, 1), 0), (3, (20, 25, 40), 0), (3, (33, 9, 7), 0), (3, (100, 50, 61), 0), (3, (190, 131, 30), 0),
    (3, (80, 80, 80), 1), (3, (130, 70, 90), 1)])
def test_default_chunk_changes_nothing(lattice, dims, precision):
    from paper_2102_09512_amd import lbm

    print("[gpu case] default tile", lattice, dims, precision, flush=True)
    f = I.smooth_random(lattice, dims, seed=11)
    states, tile, nm = [], None, dims[-1]
    for chunk in (None, 1, 5, nm):
        t = None if chunk is None else (tile[0], tile[1], min(chunk, nm))
        h = lbm.lbm_create(lattice, dims, 1.4, 0.7, 0.02, precision=precision, visc_exponent=0.76, T_ref=0.15,
                           bc=(1, 0, 0), tile=t)
        try:
            tile = tile or lbm.lbm_get_tile(h)
            assert 1 <= lbm.lbm_get_tile(h)[2] <= nm
            if precision == 1 and tile[:2] != (64, 8):
                pytest.skip("the default is a 256-thread FP32 shape here")
            lbm.lbm_init_fields(h, *f)
            lbm.lbm_step(h, 5)
            s = np.empty(lbm.lbm_state_bytes(h) // (4 if precision else 8), dtype=np.float32 if precision else np.float64)
            lbm.lbm_get_state(h, s)
            states.append(s)
        finally:
            lbm.lbm_destroy(h)
    assert np.isfinite(states[0]).all()
    assert all(np.array_equal(states[0], s) for s in states[1:])
