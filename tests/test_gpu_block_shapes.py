"""GPU parity of the general kernels that are built per block shape: every such shape with every array type, index type and
arithmetic, whole and ragged extents, rows that start anywhere, one partly filled tile and several, any mask, unaligned F."""
import numpy as np
import pytest
import torch

from paper_2406_11209_amd import synth
from parity import LINES, SHAPE, Case, route, take_wherever_possible

pytestmark = pytest.mark.gpu

SHAPES = [(16,), (32,), (64,), (4, 4), (4, 8), (8, 4), (8, 8), (8, 16), (16, 8), (16, 16), (32, 32), (2, 4, 4), (4, 4, 4),
          (4, 4, 8), (2, 8, 8), (4, 8, 8), (8, 8, 8), (2, 2, 4, 4), (2, 4, 4, 4), (4, 4, 4, 4), (2, 4, 8, 8), (2, 2, 8, 8)]
# array, working, index type: FP32 and FP64 arithmetic, none of them on a specialised family for 8x8, 16x16, 4x4x4, 8x8x8
TYPES = [("bf16", "f32", 16), ("f16", "f16", 32), ("f16", "f64", 8), ("f32", "f64", 8), ("f32", "f32", 8), ("f64", "f32", 8),
         ("f64", "f64", 16), ("f32", "bf16", 16), ("bf16", "bf16", 8), ("f64", "f64", 32)]


def extents(block, kind, g):
    """whole: multiples of the block; ragged: nothing a multiple, odd rows; small: one block, not full."""
    n = {1: 700, 2: 19, 3: 7, 4: 4}[len(block)]
    if kind == "whole":
        return tuple(b * (n if d else max(2, n - 2)) for d, b in enumerate(block))
    if kind == "ragged":
        return tuple(b * int(g.integers(2, n + 1)) + int(g.integers(1, b)) for b in block[:-1]) + (block[-1] * n + 1 + block[-1] // 2,)
    return tuple(int(g.integers(1, b + 1)) for b in block[:-1]) + (max(8, block[-1] - 1),)


def taken(block, ftype, bits):
    """Lines of 64 in FP64 work are left to the kernels for these."""
    return not (block[-1] == 64 and (ftype == "f64" or bits > 8))


def make(block, shape, dtype, ftype, bits, mask, transform, g):
    cast = {"f64": lambda a: a, "f32": lambda a: a.astype(np.float32), "bf16": synth.to_bf16_bits,
            "f16": lambda a: a.astype(np.float16)}[dtype]
    x = synth.bump_field(shape, 6, g, (2.0, 8.0)) + 0.2 + 0.01 * g.standard_normal(shape)
    x = cast(2.0 + 0.1 * x if dtype == "f16" else x)         # the check of FP16 outputs does not know subnormals
    return Case(x, None, dtype, block, bits, ftype, mask, transform=transform)


@pytest.mark.parametrize("kind", ["whole", "ragged", "small"])
@pytest.mark.parametrize("block", SHAPES, ids=["x".join(map(str, b)) for b in SHAPES])
def test_every_listed_block_shape(block, kind):
    g = np.random.Generator(np.random.PCG64(int(np.prod(block)) + len(block) + len(kind)))
    vol = int(np.prod(block))
    for n, (dtype, ftype, bits) in enumerate(TYPES):
        shape = extents(block, kind, g)
        mask = None
        if n % 3 == 1:
            mask = np.zeros(vol, dtype=bool)
            mask[g.permutation(vol)[:[1, vol // 3, vol - 2][n // 3 % 3]]] = True
            mask[0] = True
            mask = mask.reshape(block)
        case = make(block, shape, dtype, ftype, bits, mask, "haar" if n % 4 == 3 else "dct", g)
        take_wherever_possible(case.codec, SHAPE)
        exact = case.codec.kernel_name("compress", shape, dtype) != "generic"
        if not exact:
            want = SHAPE if taken(block, ftype, bits) else LINES
            assert route(case.codec, "compress", shape, dtype) == route(case.codec, "decompress", shape, dtype) == want
        N, F, _, _ = case.check_compress("A")
        case.check_decompress(N, F)
        if n % 3 == 0 or exact:
            continue                 # (a specialised kernel takes the aligned F: equal within the rounding of both only)
        # into and from F at another phase, surroundings untouched
        far_N, far_F = torch.zeros(len(N) + 2, dtype=N.dtype, device="cuda"), torch.full((F.numel() + 6,), 55, dtype=F.dtype, device="cuda")
        view = far_F[3:3 + F.numel()].view(F.shape)
        case.codec.compress(case.xA, far_N[1:-1], view)
        y = case.codec.decompress(N, F, shape, case.xA.dtype)
        far_y = case.codec.decompress(far_N[1:-1], view, shape, case.xA.dtype)
        torch.cuda.synchronize()
        assert torch.equal(view, F) and torch.equal(far_N[1:-1], N) and torch.equal(far_y, y)
        assert bool((far_F[:3] == 55).all()) and bool((far_F[-3:] == 55).all())


def test_leading_unit_dimensions_fold():
    g = np.random.Generator(np.random.PCG64(3))
    case = make((1, 1, 2, 4, 8, 8), (2, 3, 5, 9, 17, 21), "f32", "f32", 8, None, "dct", g)
    take_wherever_possible(case.codec, SHAPE)
    assert route(case.codec, "compress", case.shape, "f32") == SHAPE
    N, F, _, _ = case.check_compress("A")
    case.check_decompress(N, F)
