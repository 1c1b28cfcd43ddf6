"""The launch geometry of the diagnostics, on the host: the shapes that calls on
the device found faster, and for any box a grid that covers it, in a compiled
shape, with no more partial sums than the allocation-free scratch holds."""
import ctypes as C
import random

import pytest

from paper_2102_09512_amd import lbm


class _Grid(C.Structure):
    _fields_ = [(k, C.c_int) for k in ("bx", "by", "tiles_x", "tiles_y", "chunk", "tasks", "blocks")] + [("flat", C.c_bool)]


def _grid(dims, precision):
    f = lbm.raw()._ZN3lbm9diag_gridEiiPKl  # lbm::diag_grid(int, int, const int64_t*)
    f.restype, f.argtypes = _Grid, [C.c_int, C.c_int, C.POINTER(C.c_int64)]
    return f(len(dims), precision, (C.c_int64 * 3)(*dims, *[1] * (3 - len(dims))))


# us of a call: tiles in turn over the dies, 1024 work-groups as the aim; this choice; the form through memory
@pytest.mark.parametrize("dims,precision,tile", [
    ((100, 90, 80), 0, (64, 8, 8)),       # 142, 105, 125
    ((70, 9, 300), 0, (32, 8, 4)),        # 65, 55, 54
    ((20, 100, 100), 0, (32, 8, 3)),      # 66, 52, 58
    ((166, 213, 86), 0, (64, 8, 29)),     # 397, 304, 388
    ((268, 101, 61), 0, (32, 16, 16)),    # 241, 200, 227
    ((88, 92, 139), 0, (32, 16, 10)),     # 195, 145, 166
    ((64, 64, 64), 0, (32, 8, 4)),        # 59, 54, 63
    ((25, 168, 224), 1, (32, 16, 10)),    # 111, 77, 100
    ((256, 256, 256), 1, (64, 8, 128)),   # 868, 718, 1191
])
def test_takes_the_faster_geometry(dims, precision, tile):
    g = _grid(dims, precision)
    assert not g.flat and (g.bx, g.by, g.chunk) == tile


def test_any_box_is_covered():
    r = random.Random(4)
    for _ in range(4000):
        D = r.choice((2, 3))
        dims = tuple(max(1, int(10 ** r.uniform(0, 5 if D == 2 else 3))) for _ in range(D))
        g = _grid(dims, r.choice((0, 1)))
        assert 1 <= g.blocks <= 2048, dims
        if g.flat:
            assert g.blocks % 8 == 0, dims
            continue
        assert (g.bx, g.by) in ([(128, 1)] if D == 2 else [(64, 8), (32, 16), (32, 8)]), dims
        nm, chunks = dims[-1], -(-dims[-1] // g.chunk)
        assert 1 <= g.chunk <= nm and g.tiles_x == -(-dims[0] // g.bx), dims
        assert g.tiles_y == (1 if D == 2 else -(-dims[1] // g.by)), dims
        assert g.tasks == g.tiles_x * g.tiles_y * chunks, dims
        assert g.blocks == min(g.tasks, 2048), dims
