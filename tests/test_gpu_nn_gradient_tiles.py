"""Weight gradients where the tiles are dealt out over the work-groups
differently: fewer tiles than work-groups (one half idle), two and three tiles
per work-group with a last work-group that has fewer, both input widths, and
output layers on both sides of the eight channels that go eight to a node."""
import numpy as np
import pytest

from oracle import convnet as N

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("channels", [[5, 32, 3], [16, 32, 16], [5, 32, 32, 1], [8, 32, 8], [9, 32, 9]])
@pytest.mark.parametrize("dims", [(32, 4, 4), (64, 12, 8), (32, 20, 104), (32, 44, 100)])
def test_gradients(dims, channels):
    import torch

    from paper_2102_09512_amd import lbm

    print("[gpu case] gradient tiles", dims, channels, flush=True)
    r = np.random.default_rng(sum(dims) + channels[0])
    shape = dims[::-1]
    p = np.concatenate([np.concatenate([r.normal(0, np.sqrt(2 / (27 * i)), 27 * i * o), r.normal(0, 0.01, o)])
                        for i, o in zip(channels, channels[1:])]).astype(np.float32)
    x = r.normal(size=(channels[0],) + shape).astype(np.float32)
    t = (x + 0.3 * r.normal(size=x.shape)).astype(np.float32)
    mean, std, out = np.zeros(channels[0]), np.ones(channels[0]), np.full(channels[-1], 0.3)
    n = lbm.lbm_nn_create(channels, dims)
    try:
        lbm.lbm_nn_set_params(n, p)
        lbm.lbm_nn_set_scaling(n, mean, std, out)
        grads = []
        for _ in range(2):  # twice: a fixed order of summation
            lbm.lbm_nn_zero_grad(n)
            lbm.lbm_nn_loss_backward(n, torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda())
            grads.append(lbm.lbm_nn_get_grads(n))
    finally:
        lbm.lbm_nn_destroy(n)
    assert np.array_equal(*grads)
    _, ref = N.loss_and_grad(p.astype(np.float64), channels, x.astype(np.float64), t.astype(np.float64), mean, std,
                             store=N.bf16, out_std=out)
    g, off = grads[0].astype(np.float64), 0
    for i, o in zip(channels, channels[1:]):
        for size in (27 * i * o, o):
            a, b = g[off: off + size], ref[off: off + size]
            off += size
            # the same bf16 roundings as the reference, sums in another order (as for the whole network)
            assert a @ b / (np.linalg.norm(a) * np.linalg.norm(b)) > 0.99999
            assert np.abs(a - b).max() <= 1e-2 * np.abs(b).max()
