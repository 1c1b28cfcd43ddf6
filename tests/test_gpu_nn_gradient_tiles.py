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


@pytest.mark.parametrize("dims,layers", [((32, 4, 4), 11), ((32, 32, 64), 7)])
def test_gradient_sums_of_many_layers(dims, layers):
    """More layers than one summing launch takes, and more partials than the
    workspace holds at a time.  Small whole numbers throughout (layers that
    copy their input, 2 / (C V) a power of two): activations and their
    gradients stay below 2^8 and the sums below 2^24, so every value is exact
    in bf16 and FP32 and the gradients have to be equal."""
    import torch

    from paper_2102_09512_amd import lbm

    print("[gpu case] gradient sums", dims, layers, flush=True)
    channels = [5] + [32] * (layers - 1) + [2]
    r = np.random.default_rng(layers)
    p = []
    for i, o in zip(channels, channels[1:]):
        w = np.zeros((27, i, o))
        a, b = np.arange(i)[:, None], np.arange(o)[None, :]
        w[13] = (a == b % 5) if i == 5 else (a == b) if o == 32 else ((a + b) % 3 == 0)
        p += [w.ravel(), np.zeros(o)]
    p = np.concatenate(p).astype(np.float32)
    x = r.integers(1, 4, (5,) + dims[::-1]).astype(np.float32)
    t = x + r.integers(-4, 5, x.shape).astype(np.float32)
    mean, std, out = np.zeros(5), np.ones(5), np.ones(2)
    n = lbm.lbm_nn_create(channels, dims)
    try:
        lbm.lbm_nn_set_params(n, p)
        lbm.lbm_nn_set_scaling(n, mean, std, out)
        xd, td = torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda()
        loss = lbm.lbm_nn_loss_backward(n, xd, td)
        once = lbm.lbm_nn_get_grads(n)
        lbm.lbm_nn_loss_backward(n, xd, td, sync=False)
        total, count = lbm.lbm_nn_take_loss(n)
        twice = lbm.lbm_nn_get_grads(n)
    finally:
        lbm.lbm_nn_destroy(n)
    assert count == 1 and total == loss
    ref_loss, ref = N.loss_and_grad(p.astype(np.float64), channels, x.astype(np.float64), t.astype(np.float64), mean,
                                    std, store=N.bf16, out_std=out)
    assert abs(loss - ref_loss) <= 1e-14 * loss
    assert np.array_equal(once, ref) and np.array_equal(twice, 2 * ref)
    off = 0
    for i, o in zip(channels, channels[1:]):  # every layer takes part
        assert np.abs(ref[off: off + 27 * i * o]).max() > 0
        off += 27 * i * o + o
