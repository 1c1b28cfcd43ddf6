"""The march chunks of a batch, on the host: a box's own chunk is for a device
that it has to itself, so boxes that share the device many times over keep the
longer default chunk, and a box alone in its batch has its own."""
import ctypes as C

import pytest

from paper_2102_09512_amd import lbm


class _Tile(C.Structure):
    _fields_ = [("bx", C.c_int), ("by", C.c_int), ("chunk", C.c_int)]


def _extents(boxes):
    return (C.c_int64 * (3 * len(boxes)))(*[n for b in boxes for n in (*b, *[1] * (3 - len(b)))])


def _batch(boxes, precision):
    """(bx, by) and the boxes' chunks; the symbols are lbm::batch_shape and lbm::batch_chunks."""
    D, n, raw = len(boxes[0]), _extents(boxes), lbm.raw()
    shape, chunks = raw._ZN3lbm11batch_shapeEiiPKNS_6ExtentEi, raw._ZN3lbm12batch_chunksEiiPKNS_6ExtentEiiiPi
    shape.restype, chunks.restype = _Tile, C.c_double
    t, c = shape(D, precision, n, len(boxes)), (C.c_int * len(boxes))()
    chunks(D, precision, n, len(boxes), t.bx, t.by, c)
    return (t.bx, t.by), list(c)


def _default_chunk(box, shape):
    f = lbm.raw()._ZN3lbm13default_chunkEiPKlii
    return f(len(box), _extents([box]), *shape)


# FP64 us a step: own chunks, default chunks
@pytest.mark.parametrize("boxes", [
    [(16, 16, 16)] * 64,                    # 202, 123
    [(160, 160, 160)] * 2,                  # 1742, 1595
    [(1024, 64), (600, 1600)] * 2,          # 165, 154
    [(800, 4)],                             # D2Q9: what lbm_batch_tune times
])
def test_shared_device_keeps_default_chunks(boxes):
    shape, chunks = _batch(boxes, 0)
    assert chunks == [_default_chunk(b, shape) for b in boxes]


def test_many_small_boxes_do_not_pay_a_prologue_per_plane():
    _, chunks = _batch([(24, 24, 24)] * 48, 0)  # 354 us with one-plane chunks, 229 with these
    assert min(chunks) >= 4


@pytest.mark.parametrize("box,own", [((20, 25, 40), ((32, 8), 1)), ((32, 32, 32), ((32, 8), 1))])
def test_a_box_alone_has_its_own_chunk(box, own):
    shape, chunks = _batch([box], 0)
    assert (shape, chunks[0]) == own


def test_fp32_boxes_of_two_planes_in_flight_keep_the_chunk_they_have_alone():
    """Their rounding follows the chunk, and a batch gives lbm_step's bits."""
    for boxes in ([(64, 64, 64)] * 16, [(20, 25, 40)], [(300, 300)] * 64, [(32, 32, 32), (64, 64, 64)]):
        shape, chunks = _batch(boxes, 1)
        assert shape != (64, 8)
        assert chunks == [_default_chunk(b, shape) for b in boxes]
