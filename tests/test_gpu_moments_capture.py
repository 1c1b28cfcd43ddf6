"""lbm_moments asks for no device memory, also where its results go through a
staging buffer (pinned host memory, an address between two doubles): the call can
be captured on a handle that was initialised from device arrays, and every
replay gives the fields of that moment."""
import numpy as np
import pytest

from paper_2102_09512_amd import inputs as I

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("lattice,dims", [(2, (1, 1)), (2, (65, 9)), (3, (5, 4, 3)), (3, (33, 10, 6))])
def test_staged_moments_in_a_graph(lattice, dims, precision):
    from paper_2102_09512_amd import lbm

    print("[gpu case] captured moments", lattice, dims, precision, flush=True)
    f = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in I.smooth_random(lattice, dims, seed=6)]
    N = f[0].numel()
    pinned = [torch.zeros(a.numel(), dtype=torch.float64, pin_memory=True) for a in f]
    odd = torch.zeros(8 * N + 8, dtype=torch.uint8, device="cuda")  # one plane, 4 bytes into it
    h = lbm.lbm_create(lattice, dims, 1.4, 0.7, 0.02, precision=precision, T_ref=0.15)
    s = torch.cuda.Stream()
    try:
        torch.cuda.synchronize()
        lbm.lbm_set_stream(h, s)
        lbm.lbm_init_fields(h, *f)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            raw = lbm.raw()
            a = raw.lbm_moments(h, *[p.data_ptr() for p in pinned], lbm.LBM_DEVICE)
            b = raw.lbm_moments(h, odd.data_ptr() + 4, None, None, lbm.LBM_DEVICE)
        assert (a, b) == (0, 0), lbm.lbm_last_error()
        with torch.cuda.stream(s):
            for steps in (0, 2, 4):
                lbm.lbm_step(h, steps)  # an even number: the state stays in the captured buffer
                g.replay()
                s.synchronize()
                ref = [np.empty(tuple(x.shape)) for x in f]
                lbm.lbm_moments(h, *ref)
                for got, r in zip(pinned, ref):
                    assert np.array_equal(got.numpy(), r.ravel()), steps
                assert np.array_equal(odd.cpu().numpy()[4:4 + 8 * N].view(np.float64), ref[0].ravel()), steps
    finally:
        torch.cuda.synchronize()
        lbm.lbm_destroy(h)
