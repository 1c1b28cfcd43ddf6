"""Device allocations of the entry points that promise none, counted in the
debug library (every hipMalloc of the library): on handles that were initialised
from host arrays and so own no partial sums, lbm_diagnostics_noalloc and
lbm_moments allocate nothing, while lbm_diagnostics does, so the count can tell.
The sums are those of plain numpy."""
import ctypes as C

import numpy as np
import pytest

from paper_2102_09512_amd import build, inputs as I
from test_gpu_field_paths import _sums

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("lattice,dims,precision", [(3, (96, 40, 30), 1), (3, (5, 30, 20), 0), (2, (300, 200), 0),
                                                    (2, (20, 300), 1)])
def test_noalloc_allocates_nothing(lattice, dims, precision):
    from paper_2102_09512_amd import lbm

    print("[gpu case] counted allocations", lattice, dims, precision, flush=True)
    L = lbm._load(build.COUNTED_LIB)
    L.lbm_debug_allocations.restype = C.c_longlong
    o = lbm.lbm_default_options()
    o.precision, o.T_ref, o.visc_exponent = precision, 0.15, 0.76
    h, d = C.c_void_p(), lbm.lbm_diag()
    assert L.lbm_create(C.byref(h), lattice, (C.c_int64 * 3)(*dims, *[1] * (3 - lattice)), 1.4, 0.7, 0.02,
                        C.byref(o)) == lbm.LBM_OK
    try:
        f = [np.ascontiguousarray(a) for a in I.smooth_random(lattice, dims, seed=5)]
        f[1] += 0.03
        assert L.lbm_init_fields(h, *[a.ctypes.data for a in f], lbm.LBM_HOST) == lbm.LBM_OK
        m = [np.empty_like(a) for a in f]
        dev = [torch.empty(a.shape, dtype=torch.float64, device="cuda") for a in f]
        before = L.lbm_debug_allocations()
        assert before > 0  # the populations
        assert L.lbm_moments(h, *[a.ctypes.data for a in m], lbm.LBM_HOST) == lbm.LBM_OK
        assert L.lbm_moments(h, *[a.data_ptr() for a in dev], lbm.LBM_DEVICE) == lbm.LBM_OK
        for _ in range(2):
            assert L.lbm_diagnostics_noalloc(h, C.byref(d)) == lbm.LBM_OK
        assert L.lbm_debug_allocations() == before
        got = lbm._diag_dict(d)
        for k, v in _sums(lattice, *m, [False] * 3, 0.02, 0.76, 0.15, 2.5).items():
            # a few thousand roundings of relative size 2^-53 on sums of one sign or with a mean velocity well above
            # their scatter; the differences lose |u| / |du| <= 1e3 more
            scale = np.abs(np.asarray(v)) + 1e-10 * f[0].size
            assert np.all(np.abs(np.asarray(got[k]) - np.asarray(v)) <= 1e-11 * scale), (k, got[k], v)
        assert L.lbm_diagnostics(h, C.byref(d)) == lbm.LBM_OK
        assert L.lbm_debug_allocations() > before  # its partial sums: the count sees an allocation
        assert lbm._diag_dict(d) == got
    finally:
        torch.cuda.synchronize()
        L.lbm_destroy(h)
