"""The tuner of a batch times what it replaces: small D3Q27 boxes whose own
chunks of a plane or two take half the time of the four-plane ones keep them."""
import numpy as np
import pytest

from paper_2102_09512_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("boxes", [[(20, 25, 40)], [(12, 10, 8)] * 3])
def test_tuning_keeps_the_faster_chunks(boxes):
    from paper_2102_09512_amd import lbm

    print("[gpu case] tuned batch of small boxes", boxes, flush=True)
    hs = [lbm.lbm_create(3, d, 1.4, 0.7, 0.02, T_ref=0.15) for d in boxes]
    b = lbm.lbm_batch_create(hs)
    try:
        for h, d in zip(hs, boxes):
            lbm.lbm_init_fields(h, *I.smooth_random(3, d, seed=2))
        lbm.lbm_batch_tune(b, 20)
        # 15 us a step with the chunks chosen for the boxes (chunk 0), 29 us with four planes, in any shape
        assert lbm.lbm_batch_get_tile(b)[2] == 0
        lbm.lbm_batch_step(b, 6)
        for h, d in zip(hs, boxes):
            alone = lbm.lbm_create(3, d, 1.4, 0.7, 0.02, T_ref=0.15)
            try:
                lbm.lbm_init_fields(alone, *I.smooth_random(3, d, seed=2))
                lbm.lbm_step(alone, 6)
                m, r = [[np.empty_like(a) for a in I.smooth_random(3, d, seed=2)] for _ in range(2)]
                lbm.lbm_moments(h, *m)
                lbm.lbm_moments(alone, *r)
                for x, y in zip(m, r):
                    assert np.abs(x - y).max() <= 1e-13  # FP64 rounding of values up to 1
            finally:
                lbm.lbm_destroy(alone)
    finally:
        lbm.lbm_batch_destroy(b)
        for h in hs:
            lbm.lbm_destroy(h)
