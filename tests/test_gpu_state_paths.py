"""Device-array paths of the checkpoint calls: the kernels address the caller's
tensor directly where it is element-aligned device memory, and go through a
staging buffer otherwise.  Both must give the host path's bytes."""
import numpy as np
import pytest

from paper_2102_09512_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", [0, 1])
@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("lattice,dims", [(2, (1, 1)), (2, (130, 7)), (3, (5, 3, 2)), (3, (65, 17, 9))])
def test_state_direct_and_staged(lattice, dims, precision, layout):
    import torch

    from paper_2102_09512_amd import lbm

    print("[gpu case] state paths", lattice, dims, precision, layout, flush=True)
    dtype = torch.float64 if precision == 0 else torch.float32
    word = 8 if precision == 0 else 4
    h = lbm.lbm_create(lattice, dims, 1.4, 0.7, 0.02, precision=precision, T_ref=0.15, layout=layout)
    try:
        lbm.lbm_init_fields(h, *I.smooth_random(lattice, dims, seed=3))
        lbm.lbm_step(h, 3)
        n = lbm.lbm_state_bytes(h) // word
        host = np.empty(n, dtype=np.float64 if precision == 0 else np.float32)
        lbm.lbm_get_state(h, host)
        room = torch.zeros(n + 2, dtype=dtype, device="cuda")
        raw = lbm.raw()
        base = room.data_ptr()
        for shift in (0, word, 1):  # aligned; odd element; not element-aligned (staged)
            room.zero_()
            assert raw.lbm_get_state(h, base + shift, n * word, lbm.LBM_DEVICE) == 0
            torch.cuda.synchronize()
            got = room.cpu().numpy().view(np.uint8)
            assert np.array_equal(got[shift: shift + n * word], host.view(np.uint8))
            assert not got[:shift].any() and not got[shift + n * word:].any()
            # back in from the same place, after the state has moved on
            lbm.lbm_step(h, 1)
            assert raw.lbm_set_state(h, base + shift, n * word, lbm.LBM_DEVICE, 3) == 0
            again = np.empty_like(host)
            lbm.lbm_get_state(h, again)
            assert np.array_equal(again.view(np.uint8), host.view(np.uint8))
    finally:
        lbm.lbm_destroy(h)
