"""The default launch shape's rule, on the host: it keeps the power-of-two chunk
where sweeps on the device found the chosen shape slower, takes the finer chunk
where they found it faster, and always gives a compiled shape and a chunk within
the march axis."""
import ctypes as C
import random

import pytest

from paper_2102_09512_amd import lbm


class _Tile(C.Structure):
    _fields_ = [("bx", C.c_int), ("by", C.c_int), ("chunk", C.c_int)]


def _tile(dims, precision, caloric=False):
    f = lbm.raw()._ZN3lbm12default_tileEiiPKlb  # lbm::default_tile(int, int, const int64_t*, bool)
    f.restype, f.argtypes = _Tile, [C.c_int, C.c_int, C.POINTER(C.c_int64), C.c_bool]
    t = f(len(dims), precision, (C.c_int64 * 3)(*dims, *[1] * (3 - len(dims))), caloric)
    return t.bx, t.by, t.chunk


# us a step: base, what a rule that counts parts of a round takes
@pytest.mark.parametrize("dims,precision,base", [
    ((224, 224, 224), 0, (64, 4, 224)),    # 2120, 2525 (32 x 8 / 56)
    ((176, 176, 176), 0, (64, 4, 16)),     # 1127, 1241 (64 x 4 / 30)
    ((240, 200, 180), 0, (64, 4, 180)),    # 1661, 1924 (64 x 4 / 45)
    ((200, 150, 250), 0, (64, 4, 32)),     # 1668, 1755 (32 x 8 / 42)
    ((227, 150, 40), 0, (64, 4, 8)),       # 312, 358 (64 x 4 / 40)
    ((176, 176, 176), 1, (64, 8, 16)),     # 556, 575 (64 x 8 / 59)
    ((144, 144, 144), 1, (64, 8, 16)),     # 343, 354 (64 x 8 / 36)
    ((4888, 2248), 0, (256, 1, 32)),       # 597, 692 (256 x 1 / 29)
    ((1809, 5516), 0, (256, 1, 32)),       # 569, 649 (256 x 1 / 28)
])
def test_keeps_the_faster_base(dims, precision, base):
    assert _tile(dims, precision) == base


@pytest.mark.parametrize("dims,precision,tile", [
    ((20, 25, 40), 0, (32, 8, 1)),      # 31.4 (64 x 4 / 4), 14.6
    ((100, 100, 100), 0, (64, 4, 20)),  # 285 (64 x 4 / 32), 210
    ((800, 4), 0, (128, 1, 1)),         # 11.2 (128 x 1 / 4), 6.2
    ((300, 300), 0, (128, 1, 1)),       # 15.1 (128 x 1 / 4), 10.7
    ((190, 131, 110), 1, (64, 8, 22)),  # 346 (64 x 8 / 32), 296
])
def test_takes_the_faster_chunk(dims, precision, tile):
    assert _tile(dims, precision) == tile


def test_any_box_gets_a_compiled_shape():
    r = random.Random(3)
    for k in range(3000):
        D = r.choice((2, 3))
        dims = tuple(max(1, int(10 ** r.uniform(0, 4 if D == 2 else 2.8))) for _ in range(D))
        precision, caloric = r.choice((0, 1)), r.random() < 0.2
        bx, by, chunk = _tile(dims, precision, caloric)
        assert 1 <= chunk <= dims[-1], dims
        if D == 2:
            assert by == 1 and bx in ((128,) if caloric else (128, 256)), dims
        else:
            shapes = [(64, 4)] if caloric else [(64, 4), (32, 8)] + ([(64, 8)] if precision else [])
            assert (bx, by) in shapes, dims
