"""GPU parity of the specialised kernel families under arbitrary pruning masks: every block shape, array, working and
index type of theirs, one kept entry to all but one, whole and partly filled tiles, ragged extents, unaligned F."""
import numpy as np
import pytest
import torch

from paper_2406_11209_amd import api, synth
from parity import MASKED, SHAPE, TILED, Case, route, take_wherever_possible

pytestmark = pytest.mark.gpu

# shapes: ragged slow extents and a partly filled last tile with whole rows; rows with a partial last block; whole tiles
SHAPES = {(8, 8): [(21, 72), (19, 1030), (16, 1024)], (4, 4, 4): [(5, 6, 28), (9, 13, 262), (4, 8, 512)],
          (16, 16): [(35, 288), (21, 78), (32, 512)], (4, 16, 16): [(9, 20, 48), (6, 33, 150), (8, 16, 128)],
          (8, 8, 8): [(9, 17, 24), (17, 9, 70), (8, 16, 128)], (16, 16, 16): [(20, 37, 48), (17, 16, 70), (16, 16, 64)]}
TYPES = {(8, 8): "f32 f32 8,f32 f16 16,f32 f32 32,bf16 f32 8,f16 bf16 8,f64 f64 8,f64 f64 16,f64 f64 32,f64 f32 8,f64 f32 16",
         (4, 4, 4): "f32 f32 8,f32 f32 16,f32 f32 32,f64 f64 8,f64 f64 16,f64 f64 32,f64 f32 8,f64 bf16 16",
         (16, 16): "f32 f32 8,f32 f32 16,f32 f32 32,bf16 f32 8,f16 f32 8,f64 f64 8,f64 f64 16,f64 f64 32,f64 f32 8",
         (4, 16, 16): "f32 f32 8,f32 f32 16,f32 f32 32,f16 f32 8,f64 f64 8,f64 f64 16,f64 f64 32,f64 f32 8",
         (8, 8, 8): "f32 f32 8,f32 f32 16,f32 f32 32,bf16 f32 8,f16 f32 8,f64 f64 8,f64 f64 16,f64 f64 32,f64 f32 8",
         (16, 16, 16): "f32 f32 8,f32 f32 16,f32 f32 32,f64 f64 8,f64 f64 16,f64 f64 32,f64 f32 8"}
ROWS = [(block, *t.split()) for block, types in TYPES.items() for t in types.split(",")]


def kind(block, dtype, ftype, bits):
    """FP64 arrays in FP64 work in the smaller blocks are left to the kernels per block shape."""
    return SHAPE if dtype == "f64" and block in ((8, 8), (4, 4, 4)) and (ftype == "f64" or bits > 8) else MASKED


def random_mask(block, kept, g):
    vol = int(np.prod(block))
    m = np.zeros(vol, dtype=bool)
    m[g.permutation(vol)[:kept]] = True
    return m.reshape(block)


@pytest.mark.parametrize("transform", ["dct", "haar"])
@pytest.mark.parametrize("block,dtype,ftype,bits", ROWS, ids=["%s-%s-%s-i%s" % r for r in ROWS])
def test_any_mask_on_the_specialised_families(block, dtype, ftype, bits, transform):
    bits, vol = int(bits), int(np.prod(block))
    g = np.random.Generator(np.random.PCG64(vol + bits + len(dtype)))
    cast = {"f64": lambda a: a, "f32": lambda a: a.astype(np.float32), "bf16": synth.to_bf16_bits,
            "f16": lambda a: a.astype(np.float16)}[dtype]
    for shape, kept in zip(SHAPES[block] + SHAPES[block][:2], (vol // 4, vol - 1, 19, 1, vol // 2)):
        x = cast(synth.bump_field(shape, 6, g, (2.0, 8.0)) + 0.2 + 0.01 * g.standard_normal(shape))
        mask = random_mask(block, kept, g)
        case = Case(x, None, dtype, block, bits, ftype, mask, transform=transform)
        take_wherever_possible(case.codec, MASKED)
        want = kind(block, dtype, ftype, bits)
        if want == SHAPE:
            take_wherever_possible(case.codec, SHAPE)
        assert route(case.codec, "compress", shape, dtype) == route(case.codec, "decompress", shape, dtype) == want
        N, F, _, _ = case.check_compress("A")
        case.check_decompress(N, F)
        # the same into and from F one block on, which is another phase unless a block is whole 16-byte pieces
        far_N, far_F = torch.zeros(len(N) + 2, dtype=N.dtype, device="cuda"), torch.full((len(F) + 2, kept), 55, dtype=F.dtype, device="cuda")
        case.codec.compress(case.xA, far_N[1:-1], far_F[1:-1])
        y = case.codec.decompress(N, F, shape, case.xA.dtype)
        far_y = case.codec.decompress(far_N[1:-1], far_F[1:-1], shape, case.xA.dtype)
        torch.cuda.synchronize()
        assert torch.equal(far_F[1:-1], F) and torch.equal(far_N[1:-1], N) and torch.equal(far_y, y)
        assert bool((far_F[0] == 55).all()) and bool((far_F[-1] == 55).all()) and float(far_N[0]) == 0.0 == float(far_N[-1])
        # the tiled kernels see the same: their reconstruction of the same {N, F}
        slow = Case(x, None, dtype, block, bits, ftype, mask, api.PBZ_PATH_GENERIC, transform=transform)
        assert route(slow.codec, "decompress", shape, dtype) == TILED
        slow.check_decompress(N, F)
