"""Which kernels a call of a specialised family goes to (host only): settings that the kernels per block shape took while the family's own were the faster
ones, and the same settings on the other side of each line."""
import numpy as np
import pytest

from paper_2406_11209_amd.api import Codec
from parity import EXACT, SHAPE, TILED, route

# direction, block, array, work, index bits, transform, [(shape, kernels)]
LINES = [("decompress", (8, 8, 8), "f64", "f64", 8, "dct", [((4, 3, 1390), EXACT), ((48, 139, 76), EXACT), ((64, 184, 250), EXACT), ((64, 248, 250), SHAPE)]),    # 1.2-1.9 of the time up to 2 Mi
         ("decompress", (8, 8, 8), "f64", "f64", 8, "haar", [((224, 146, 13), EXACT), ((64, 248, 250), SHAPE)]),
         ("decompress", (8, 8, 8), "f64", "f64", 32, "dct", [((64, 248, 250), EXACT), ((64, 400, 250), SHAPE)]),
         ("decompress", (8, 8, 8), "f32", "f32", 32, "dct", [((232, 816, 24), EXACT), ((320, 816, 16), SHAPE), ((648, 312, 23), EXACT)]),
         ("decompress", (8, 8, 8), "f32", "f32", 16, "dct", [((232, 816, 24), SHAPE)]),
         ("decompress", (8, 8, 8), "bf16", "bf16", 8, "haar", [((688, 384, 24), EXACT), ((1400, 384, 8), SHAPE)]),
         ("decompress", (16, 16), "f64", "f64", 32, "dct", [((5401, 1336), EXACT), ((40000, 120), SHAPE), ((34144, 224), EXACT)]),
         ("decompress", (16, 16), "f64", "f32", 32, "dct", [((34144, 226), EXACT)]),
         ("decompress", (16, 16), "f64", "f64", 8, "dct", [((13264, 1114), EXACT), ((40000, 150), SHAPE)]),
         ("decompress", (16, 16), "f64", "f64", 16, "dct", [((12640, 1580), EXACT), ((40000, 190), SHAPE)]),
         ("decompress", (16, 16), "f32", "f32", 8, "haar", [((148560, 96), EXACT), ((148560, 64), SHAPE)]),
         ("decompress", (16, 16), "f32", "f32", 8, "dct", [((148560, 128), EXACT), ((148560, 96), SHAPE)]),
         ("decompress", (8, 8), "f16", "f16", 8, "dct", [((6640, 1294), EXACT), ((15651, 322), EXACT), ((20000, 300), SHAPE)]),
         ("decompress", (8, 8), "f32", "f32", 8, "dct", [((20104, 216), EXACT), ((40000, 160), SHAPE)]),
         ("decompress", (8, 8), "f32", "f32", 8, "haar", [((40000, 160), EXACT), ((60000, 72), SHAPE)]),
         ("decompress", (8, 8), "f32", "f32", 16, "haar", [((16417, 191), EXACT), ((23974, 188), EXACT), ((79266, 107), SHAPE)]),     # 1.1-1.4
         ("decompress", (8, 8), "f32", "f32", 16, "dct", [((126787, 178), SHAPE)]),
         ("compress", (16, 16), "f64", "f64", 8, "haar", [((28083, 1538), EXACT), ((100000, 190), SHAPE)]),
         ("compress", (8, 8), "f32", "f32", 8, "dct", [((4568, 1990), EXACT), ((30000, 398), SHAPE)]),
         ("compress", (4, 4, 4), "f64", "f64", 32, "dct", [((60, 140, 1502), EXACT), ((60, 600, 226), SHAPE)])]


@pytest.mark.parametrize("line", LINES, ids=lambda line: "-".join(map(str, line[:6])))
def test_where_the_lines_lie(line):
    op, block, dtype, ftype, bits, transform, calls = line
    codec = Codec(block, ftype, bits, None, transform)
    assert [(shape, route(codec, op, shape, dtype)) for shape, _ in calls] == calls


# the same between the kernels per block shape and the tiled ones, with how many of a block's coefficients are kept
SHAPE_LINES = [((4, 8, 8), "f64", "f32", 16, "dct", 4, [((10, 11, 86), TILED), ((272, 429, 2), TILED), ((10, 11, 86 * 128), SHAPE)]),    # 1.05-1.23 of the time
               ((4, 8, 8), "f64", "f32", 16, "dct", 2, [((10, 11, 86), SHAPE)]),
               ((4, 8, 8), "f32", "f32", 8, "dct", 4, [((48, 24, 80), TILED), ((48, 24, 77), SHAPE)]),
               ((32, 32), "f64", "f32", 8, "dct", 4, [((646, 102), TILED), ((646, 101), SHAPE)]),
               ((32, 32), "f64", "f32", 8, "dct", 2, [((646, 102), SHAPE)]),
               ((32, 32), "f64", "f32", 8, "haar", 2, [((646, 102), TILED)]),
               ((32, 32), "f64", "f64", 16, "haar", 4, [((760, 380), TILED)]),
               ((32, 32), "f64", "f64", 16, "dct", 4, [((760, 380), SHAPE)]),
               ((32, 32), "f32", "f32", 8, "dct", 4, [((752, 40), TILED), ((752, 41), SHAPE), ((2000, 1000), SHAPE)]),                     # 1.06-1.18
               ((32, 32), "bf16", "f32", 16, "haar", 4, [((306, 312), TILED), ((306, 311), SHAPE), ((2000, 1000), SHAPE)]),                # 1.2-1.36
               ((32,), "f64", "f64", 32, "haar", 1, [((2350099,), TILED), ((3300099,), SHAPE)]),
               ((32,), "f32", "f32", 32, "haar", 1, [((24316,), TILED), ((2220256,), TILED), ((24317,), SHAPE)]),                          # 1.2-1.4
               ((32,), "f64", "f64", 32, "dct", 1, [((24318,), TILED), ((1 << 21,), SHAPE)])]


@pytest.mark.parametrize("line", SHAPE_LINES, ids=lambda line: "-".join(map(str, line[:6])))
def test_where_decompressed_rows_of_whole_pieces_go(line):
    block, dtype, ftype, bits, transform, share, calls = line
    mask = np.arange(int(np.prod(block))).reshape(block) % share == 0 if share > 1 else None
    codec = Codec(block, ftype, bits, mask, transform)
    assert [(shape, route(codec, "decompress", shape, dtype)) for shape, _ in calls] == calls


def test_lines_of_32_with_32_bit_indices():
    for ftype, transform in (("f32", "dct"), ("f64", "haar")):
        codec = Codec((32,), ftype, 32, None, transform)
        for n, where in ((2 << 20, SHAPE), ((2 << 20) + 32, TILED), ((3 << 20) - 32, TILED), (3 << 20, SHAPE)):
            assert route(codec, "compress", (n,), ftype) == where
